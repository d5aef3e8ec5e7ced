// Host-side helpers shared by the C-ABI translation units: error reporting, argument checks,
// per-step scalars, and the objects that assemble kernel launches over tensor lists.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cmath>
#include <initializer_list>
#include <cstdint>
#include <vector>

#include "zi_internal.h"
#include "zi_checks.h"
#include "zi_plan.h"

static_assert(zi::host::kPlanMaxSegmentsPerUse == zi::kMaxStepDesc, "a packed slot use must fit one fused-step launch");

namespace zi {
namespace host {

#define ZI_HIP(call)                                                                                  \
    do {                                                                                              \
        hipError_t e_ = (call);                                                                       \
        if (e_ != hipSuccess) {                                                                       \
            (void)hipGetLastError(); /* do not leave a sticky error for the caller's next HIP call */ \
            return ::zi::host::fail(ZI_ERR_HIP, "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), __FILE__, __LINE__); \
        }                                                                                             \
    } while (0)

// What kind of memory an address is: 0 device (whose, in *device), 1 page-locked host, 2 ordinary host, -1 anything
// else, -2 if the HIP runtime cannot answer (no usable device).
inline int memory_kind(const void* p, int* device = nullptr)
{
    hipPointerAttribute_t attr{};
    const hipError_t pe = hipPointerGetAttributes(&attr, p);
    if (pe != hipSuccess) {
        (void)hipGetLastError();
        return pe == hipErrorInvalidValue ? 2 : -2;      // older runtimes report unregistered memory this way
    }
    if (device) *device = attr.device;
    if (attr.type == hipMemoryTypeDevice) return 0;
    if (attr.type == hipMemoryTypeHost) return 1;
    if (attr.type == hipMemoryTypeUnregistered) return 2;
    return -1;
}

// A kernel is about to read or write `bytes` at p: both ends must be memory the GPU can reach (device
// or page-locked host).  An ordinary host pointer here would be a GPU memory fault, not an error code.
// Device allocations that have been looked up are remembered for the rest of the call, so a list of
// thousands of views into a few allocations costs a few queries, not thousands.
struct PointerChecker {
    struct Range { uintptr_t lo, hi; };
    Range known[8] = {};
    int n_known = 0, next = 0;

    // Whether the array lies in an allocation that has been looked up.
    bool covers(const void* p, size_t bytes) const
    {
        for (int i = 0; i < n_known; ++i)
            if (lies_within(p, bytes, known[i].lo, known[i].hi)) return true;
        return false;
    }

    zi_status check(const void* p, size_t bytes, int tensor, const char* name)
    {
        if (!p || bytes == 0 || covers(p, bytes)) return ZI_OK;
        hipDeviceptr_t base = nullptr;
        size_t size = 0;
        bool inside = false;
        if (hipMemGetAddressRange(&base, &size, const_cast<void*>(p)) == hipSuccess && size > 0) {
            const uintptr_t blo = reinterpret_cast<uintptr_t>(base);
            inside = lies_within(p, bytes, blo, blo + size);
        } else {
            (void)hipGetLastError();
        }
        if (wraps_around(p, bytes)) return fail(ZI_ERR_INVALID_ARG, "tensor %d: %s (%zu bytes) is no array", tensor, name, bytes);
        // one allocation is one kind of memory: its first byte speaks for all of it
        const void* ends[2] = {p, static_cast<const char*>(p) + bytes - 1};
        for (int i = 0; i < (inside ? 1 : 2); ++i) {
            const int k = memory_kind(ends[i]);
            if (k == -2) return fail(ZI_ERR_HIP, "no usable HIP device (pointer query failed)");
            if (k != 0 && k != 1)
                return fail(ZI_ERR_INVALID_ARG, "tensor %d: %s (%zu bytes) is not device or page-locked host memory",
                            tensor, name, bytes);
        }
        if (inside) {
            const uintptr_t blo = reinterpret_cast<uintptr_t>(base);
            known[next] = {blo, blo + size};
            next = (next + 1) % 8;
            if (n_known < 8) ++n_known;
        }
        return ZI_OK;
    }
};

inline zi_status check_kernel_visible(const void* p, size_t bytes, int tensor, const char* name)
{
    PointerChecker c;
    return c.check(p, bytes, tensor, name);
}

// Number of leading elements (0..63) the step handles one by one before its vector body.  Any value
// is legal: the body's vector accesses need only element alignment.  The choice decides how much of
// the body's traffic starts on a 128-byte line (a wavefront's run then covers whole lines) and,
// failing that, on a lane-vector boundary (16 bytes for fp32, 8 for the 2-byte arrays); arrays are
// weighted by the bytes they move per element (p, m, v: 8; g, p_lp: 2).
// Arrays at one common offset have exactly one head that puts all of them on lines: it has the highest score,
// and taking it at once costs 3 ns instead of 200, which a list pays once per tensor.
inline int choose_head(const void* p, const void* m, const void* v, const void* g, const void* p_lp)
{
    const uintptr_t common = (0 - reinterpret_cast<uintptr_t>(g) / 2) % 64;
    bool all_lines = !p_lp || (reinterpret_cast<uintptr_t>(p_lp) / 2 + common) % 64 == 0;
    for (const void* x : {p, m, v}) all_lines = all_lines && (reinterpret_cast<uintptr_t>(x) / 4 + common) % 32 == 0;
    if (all_lines) return (int)common;
    int best_h = 0, best = -1;
    for (int h = 0; h < 64; ++h) {
        int score = 0;
        for (const void* x : {p, m, v}) {
            const uintptr_t i = reinterpret_cast<uintptr_t>(x) / 4 + (uintptr_t)h;
            score += 8 * (i % 32 == 0 ? 4 : i % 4 == 0 ? 1 : 0);
        }
        for (const void* x : {g, (const void*)p_lp}) {
            if (!x) continue;
            const uintptr_t i = reinterpret_cast<uintptr_t>(x) / 2 + (uintptr_t)h;
            score += 2 * (i % 64 == 0 ? 4 : i % 4 == 0 ? 1 : 0);
        }
        if (score > best) { best = score; best_h = h; }
    }
    return best_h;
}

// Tensors of at least this many tiles (2^22 elements, some 20 microseconds of HBM time) are launched
// alone; shorter ones share launches of up to kMaxStepDesc tensors.  StepIssuer::expect says which lists go to
// adamw_list_kernel instead: those of more than kMaxListDesc tensors as they are, and shorter ones by what they consist of.
#ifndef ZI_SOLO_TILES
#define ZI_SOLO_TILES 8192
#endif
constexpr int64_t kSoloTiles = ZI_SOLO_TILES;

// Whether a launch that need not wait for the one in front of it may say so: not while the stream is captured, nor
// where that cannot be told (the query fails for the null stream while another stream is captured; launches do not).
inline bool may_overlap(hipStream_t stream)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) == hipSuccess) return capture == hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

// Whether what is launched on the stream now may run again later, with the same arguments.  (The null stream cannot be
// captured; of any other stream that the query refuses it is assumed.)
inline bool is_captured(hipStream_t stream)
{
    if (!stream) return false;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) == hipSuccess) return capture != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// A call on one tensor, as launch_step_one takes it: false if it is another call, or one on more quads than StepOne counts.
inline bool one_tensor(const zi_tensor* t, int32_t n_tensors, const zi::StepConsts& c, bool l2,
                       const zi_norm_result* d_norm, zi::StepOne& a)
{
    const zi_tensor* one = nullptr;
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (t[i].numel <= 0) continue;
        if (one) return false;
        one = &t[i];
    }
    if (!one || one->numel > (int64_t)(zi::kFineMostTiles - 1) * zi::kStepTileElems) return false;
    const int64_t h = choose_head(one->p, one->m, one->v, one->g, one->p_lp), head = h < one->numel ? h : one->numel;
    a.p_body = (float*)one->p + head;
    a.m_body = (float*)one->m + head;
    a.v_body = (float*)one->v + head;
    a.g_body = (const uint16_t*)one->g + head;
    a.lp_body = one->p_lp ? (uint16_t*)one->p_lp + head : nullptr;
    a.nquad = (uint32_t)((one->numel - head) / zi::kQuad);
    a.head = (uint8_t)head;
    a.tail = (uint8_t)(one->numel - head - (int64_t)a.nquad * zi::kQuad);
    set_scalars(a, c, l2, d_norm);
    return true;
}

// Every tensor's five arrays begin the same number of elements (less than 2^32, its end included) behind the
// first tensor's, and all have a copy or none.  Sets the first tensor's addresses.
template <typename Flat>
inline bool is_flat(const zi_tensor* t, int32_t n_tensors, Flat& flat)
{
    const zi_tensor* f = nullptr;
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (t[i].numel <= 0) continue;
        if (!f) f = &t[i];
        const auto bytes = [](const void* x, const void* from) { return reinterpret_cast<uintptr_t>(x) - reinterpret_cast<uintptr_t>(from); };
        const uintptr_t at = bytes(t[i].p, f->p);
        if (at % 4 || at / 4 + (uintptr_t)t[i].numel > 0xFFFFFFFFull) return false;
        if (bytes(t[i].m, f->m) != at || bytes(t[i].v, f->v) != at || bytes(t[i].g, f->g) != at / 2) return false;
        if (!t[i].p_lp != !f->p_lp || (f->p_lp && bytes(t[i].p_lp, f->p_lp) != at / 2)) return false;
    }
    flat.p = (float*)f->p;
    flat.m = (float*)f->m;
    flat.v = (float*)f->v;
    flat.g = (const uint16_t*)f->g;
    flat.lp = (uint16_t*)f->p_lp;
    return true;
}

// What a launch over n tensors looks its tensors up in, once they are in.
template <typename Args>
inline void finish_starts(Args& a, int32_t n)
{
    for (int32_t i = n; i < Args::kMax; ++i) a.first_tile[i] = 0xFFFFFFFFu;
    for (int i = 0; i < Args::kGroups; ++i) a.group_start[i] = a.first_tile[i * Args::kGroup];
}

// Makes a tensor the n-th of a flat list, from tile `first` of the launch; returns its tiles.
template <typename Flat>
inline uint32_t add_flat(Flat& a, int32_t n, uint32_t first, const float* p, int h, int64_t numel)
{
    const int64_t head = h < numel ? h : numel, nquad = (numel - head) / zi::kQuad;
    const int64_t tiles = (nquad + zi::kStepTileQuads - 1) / zi::kStepTileQuads;
    a.t[n] = {(uint32_t)(p + head - a.p), (uint32_t)nquad};
    a.head[n] = (uint8_t)head;
    a.tail[n] = (uint8_t)(numel - head - nquad * zi::kQuad);
    a.first_tile[n] = first;
    return tiles < 1 ? 1u : (uint32_t)tiles;
}

// A call on 2 to FlatFew::kMax tensors of kFewElems elements in all that are views at the same places of five flat buffers:
// fills the launch's arguments and returns its tiles, 0 if it is another call.
inline uint32_t few_short_tensors(const zi_tensor* t, int32_t n_tensors, const zi::StepConsts& c, const zi_norm_result* d_norm,
                                  zi::FlatFew& a)
{
    int32_t n = 0;
    int64_t total = 0;
    for (int32_t i = 0; i < n_tensors && n <= zi::FlatFew::kMax && total <= zi::kFewElems; ++i) {
        n += t[i].numel > 0;
        total += t[i].numel < zi::kFewElems ? t[i].numel : zi::kFewElems + 1;
    }
    if (n < 2 || n > zi::FlatFew::kMax || total > zi::kFewElems || !is_flat(t, n_tensors, a)) return 0;
    a.c = c;
    a.d_norm = d_norm;
    uint32_t tiles = 0;
    n = 0;
    for (int32_t i = 0; i < n_tensors; ++i)
        if (t[i].numel > 0)
            tiles += add_flat(a, n++, tiles, (const float*)t[i].p, choose_head(t[i].p, t[i].m, t[i].v, t[i].g, t[i].p_lp), t[i].numel);
    finish_starts(a, n);
    return tiles;
}

// Issues the fused step over a list of device-resident segments.
struct StepIssuer {
    zi::StepArgs args{};
    uint32_t tiles = 0;
    int dt;
    bool l2;
    hipStream_t stream;
    int64_t launches = 0;
    // Planning mode (zi_plan_step): with a sink set nothing is launched; every descriptor of every
    // launch is recorded instead.  `cur_tensor` is the caller's index of the tensor being added.
    std::vector<zi_step_plan_item>* plan = nullptr;
    int32_t cur_tensor = -1;
    int32_t tensor_of[zi::FlatArgs::kMax] = {};
    // Lists of more than kMaxListDesc tensors (expect()): launches of many, whatever their length, in `list`, or in
    // `flat` if the tensors are short and all at the same places of five flat buffers; those also from kMaxStepDesc
    // tensors on, which are one launch then instead of two or more (step alone, us: 40 tensors of 1000 elements 6.3 ->
    // 3.5, 60 of 3.0e4 13.1 -> 10.2, 48 of 2.6e5 69.4 -> 66.6; one launch either way, 24 of 1.0e5 13.0 / 13.4).  Four times as many to a launch
    // save 3 us each time, and twice as many entries in the lookup cost every workgroup some 4%.  Step alone, us, list /
    // flat: 200 tensors of 2e4 elements 35.3 / 25.3, 1000 of 1e5 512 / 480, 288 of 2.6e5 361 / 352, 288 of 1.0e6
    // 1368 / 1427, 72 of 4.2e6 1363 / 1420: the line is drawn at an average of 5 * 2^16.  In fine tiles, with copies, the lookup costs less:
    // 200 of 5e5 450 / 438, a decoder's 144 at hidden size 768 375 / 370, 288 of 1.0e6 1257 / 1257, without copies 90 of 9e5 332 / 335:
    // lists that are several launches either way have the line at 2^20.
    static constexpr int64_t kFlatAverage = 5 << 16, kFlatCopiesAverage = 1 << 20;
    // Shorter lists with several long tensors among few short ones, as a few layers of a decoder are, take `list` too: a launch
    // of its own for every long tensor pays a start and an end each time, which shows up to 2^25 elements on average, and beyond
    // that the longer lookup does.  Step alone, us, own launches / list: 2 tensors of 5e6 50.4 / 47.6, 8 of 5e6 198 / 180, 30 of 1e7
    // 1369 / 1323, 8 of 3e7 1074 / 1056, 30 of 3e7 4000 / 4003, 24 of 5e7 5235 / 5250, 48 of 6.7e7 14120 / 14385; a decoder's tensors at
    // hidden size 1024, 4 layers 246 / 225, 2048, 1 layer 238 / 225, 4096, 1 layer 918 / 904, 8192, 1 layer 3490 / 3517.
    static constexpr int64_t kListAverage = (int64_t)1 << 25;
    enum Kind { kFew, kList, kFlat };
    Kind kind = kFew;
    zi::ListArgs list;
    zi::FlatArgs flat;

    // What the list will be, before the first add(): decides how many tensors share a launch.
    void expect(const zi_tensor* t, int32_t n_tensors)
    {
        int64_t n = 0, n_long = 0, total = 0;
        bool copies = false;
        for (int32_t i = 0; i < n_tensors; ++i) {
            n += t[i].numel > 0;
            copies |= t[i].numel > 0 && t[i].p_lp;
            n_long += t[i].numel >= kSoloTiles * zi::kStepTileElems;
            total += t[i].numel;
        }
        if (n < 2) return;
        const bool short_and_flat = n > zi::kMaxStepDesc && total / n <= (copies && n > zi::kMaxListDesc ? kFlatCopiesAverage : kFlatAverage) &&
                                    is_flat(t, n_tensors, flat);
        const bool middling = n_long >= 2 && n_long >= n / 8 && total / n <= kListAverage;
        if (!short_and_flat && !middling && n <= zi::kMaxListDesc) return;
        kind = short_and_flat ? kFlat : kList;
        list.c = flat.c = args.c;
        list.d_norm = flat.d_norm = args.d_norm;
    }

    int32_t max_desc() const { return kind == kFlat ? zi::FlatArgs::kMax : kind == kList ? zi::kMaxListDesc : zi::kMaxStepDesc; }

    StepIssuer(const zi::StepConsts& c, const zi_norm_result* d_norm, int dt_, bool l2_, hipStream_t s)
        : dt(dt_), l2(l2_), stream(s)
    {
        args.c = c;
        args.d_norm = d_norm;
        reset();
    }

    void reset()
    {
        args.n_desc = 0;
        tiles = 0;
        for (uint32_t& f : args.first_tile) f = 0xFFFFFFFFu;
    }

    // The launches of one call touch different tensors, so they may overlap; only the call as a whole has its
    // place in the stream.  Launches are held back by one: the first and the last are ordinary ones (the first
    // waits for everything before the call, the last for every launch of it, so whatever waits for the
    // last waits for all), those between them start as soon as workgroups of the launch before run out, instead of
    // after its last workgroup and a cache flush.  That gains 1 us a launch where the launches are short and costs 10
    // where two long ones meet, each of which alone walks its arrays in order (step alone, us, ordinary / overlapping:
    // launches of 4e6 elements 533 / 516 in all, of 1.7e7 368 / 365, of 6.4e7 1396 / 1431, of 2.7e8 14170 / 14375):
    // both have to be of kOverlapTiles or less.  Under capture all stay ordinary.
    static constexpr uint32_t kOverlapTiles = 1u << 15;
    uint32_t last_tiles = 0;          // of the launch issued last
    zi::StepArgs held;
    zi::ListArgs held_list;
    zi::FlatArgs held_flat;
    uint32_t held_tiles = 0;
    Kind held_kind = kFew;

    hipError_t issue_held(bool last)
    {
        if (held_tiles == 0) return hipSuccess;
        const bool any_order = !last && launches > 0 && held_tiles <= kOverlapTiles && last_tiles <= kOverlapTiles && may_overlap(stream);
        ++launches;
        const uint32_t n = last_tiles = held_tiles;
        held_tiles = 0;
        return held_kind == kFlat   ? zi::launch_step_flat(held_flat, n, dt, l2, any_order, stream)
               : held_kind == kList ? zi::launch_step_list(held_list, n, dt, l2, any_order, stream)
                                    : zi::launch_step_wide(held, n, dt, l2, any_order, stream);
    }

    void planned(int32_t tensor, int32_t head, int64_t first, int64_t end, bool alone)
    {
        plan->push_back({tensor, head, end - first, first, (int32_t)launches, alone ? 1 : 0});
    }

    hipError_t launch(const zi::StepArgs& a, uint32_t n_tiles, const int32_t* tensors)
    {
        if (plan) {
            for (int32_t i = 0; i < a.n_desc; ++i)
                planned(tensors[i], a.t[i].head, a.t[i].first_tile, i + 1 < a.n_desc ? a.t[i + 1].first_tile : n_tiles,
                        a.n_desc == 1);
            ++launches;
            return hipSuccess;
        }
        const hipError_t e = issue_held(false);
        held = a;
        held_tiles = n_tiles;
        held_kind = kFew;
        return e;
    }

    template <typename Args>
    hipError_t launch_list(Args& a, Args& into)
    {
        const int32_t n = args.n_desc;
        if (plan) {
            for (int32_t i = 0; i < n; ++i)
                planned(tensor_of[i], kind == kFlat ? flat.head[i] : list.t[i].head, a.first_tile[i],
                        i + 1 < n ? a.first_tile[i + 1] : tiles, n == 1);
            ++launches;
            return hipSuccess;
        }
        const hipError_t e = issue_held(false);
        finish_starts(a, n);
        into = a;
        held_tiles = tiles;
        held_kind = kind;
        return e;
    }

    hipError_t close()       // the launch being assembled is complete
    {
        hipError_t e = hipSuccess;
        if (args.n_desc > 0)
            e = kind == kFlat   ? launch_list(flat, held_flat)
                : kind == kList ? launch_list(list, held_list)
                                : launch(args, tiles, tensor_of);
        reset();
        return e;
    }

    hipError_t flush()       // end of the call
    {
        const hipError_t e = close();
        return e != hipSuccess ? e : issue_held(true);
    }

    hipError_t add(float* p, float* m, float* v, const uint16_t* g, uint16_t* p_lp, int64_t numel)
    {
        if (numel <= 0) return hipSuccess;
        zi::StepDesc d{};
        const int h = choose_head(p, m, v, g, p_lp);
        d.head = (int32_t)(h < numel ? h : numel);
        d.p_body = p + d.head; d.m_body = m + d.head; d.v_body = v + d.head; d.g_body = g + d.head;
        d.lp_body = p_lp ? p_lp + d.head : nullptr;
        d.numel = numel;
        const int64_t nquad = (numel - d.head) / zi::kQuad;
        int64_t nt = (nquad + zi::kStepTileQuads - 1) / zi::kStepTileQuads;
        if (nt < 1) nt = 1;                       // the first tile also owns the unaligned ends
        if (nt > 0x7FFFFFFF) return hipErrorInvalidValue;
        d.nquad = nquad;
        d.n_tiles = (uint32_t)nt;
        if (kind != kFew ? nquad > 0xFFFFFFFFll : nt >= kSoloTiles) {      // a launch of its own: no tensor lookup in the kernel
            zi::StepArgs solo{};
            solo.c = args.c;
            solo.d_norm = args.d_norm;
            solo.n_desc = 1;
            for (uint32_t& f : solo.first_tile) f = 0xFFFFFFFFu;
            d.first_tile = 0;
            solo.first_tile[0] = 0;
            solo.t[0] = d;
            return launch(solo, (uint32_t)nt, &cur_tensor);
        }
        if (args.n_desc == max_desc() || (uint64_t)tiles + (uint64_t)nt > 0x7FFFFFFFull) {
            hipError_t e = close();
            if (e != hipSuccess) return e;
        }
        if (kind != kFew) {
            const int32_t n = args.n_desc++;
            const int64_t tail = numel - d.head - nquad * zi::kQuad;
            if (kind == kFlat) {
                flat.t[n] = {(uint32_t)(d.p_body - flat.p), (uint32_t)nquad};
                flat.head[n] = (uint8_t)d.head;
                flat.tail[n] = (uint8_t)tail;
                flat.first_tile[n] = tiles;
            } else {
                list.t[n] = {d.p_body, d.m_body, d.v_body, d.g_body, d.lp_body, (uint32_t)nquad, (uint16_t)d.head, (uint16_t)tail};
                list.first_tile[n] = tiles;
            }
            tensor_of[n] = cur_tensor;
            tiles += (uint32_t)nt;
            return hipSuccess;
        }
        d.first_tile = tiles;
        args.first_tile[args.n_desc] = tiles;
        tensor_of[args.n_desc] = cur_tensor;
        args.t[args.n_desc++] = d;
        tiles += (uint32_t)nt;
        return hipSuccess;
    }
};

// Issues copies of 2-byte segments between device and page-locked host memory (link_copy_kernel).
struct CopyIssuer {
    zi::CopyArgs args{};
    hipStream_t stream;

    CopyIssuer(hipStream_t s, uint32_t* flags, uint32_t serial) : stream(s)
    {
        args.flags = flags;
        args.serial = serial;
    }
    hipError_t flush()
    {
        if (args.n_segs == 0) return hipSuccess;
        const hipError_t e = zi::launch_link_copy(args, stream);
        args.n_segs = args.n_blocks = 0;
        return e;
    }
    // `flag`: index of the first block's flag (unused without flags).
    hipError_t add(const uint16_t* src, uint16_t* dst, int64_t elems, uint32_t flag)
    {
        if (elems <= 0) return hipSuccess;
        if (args.n_segs == (uint32_t)zi::kMaxCopySegs)
            if (const hipError_t e = flush(); e != hipSuccess) return e;
        args.t[args.n_segs++] = {src, dst, elems, args.n_blocks, flag};
        const int64_t block = args.flags ? zi::kCopyBlockElems : zi::kCopyPieceElems;
        args.n_blocks += (uint32_t)((elems + block - 1) / block);
        return hipSuccess;
    }
};

// Issues the step over segments in page-locked host memory (adamw_link_kernel, adamw_link_flat_kernel), kLinkTilesPerLaunch
// tiles to a launch at most.  Long segments are cut where a launch is full, a multiple of 512 elements into the segment's
// body; those of flat lists are not cut, and a list with one that is longer than a launch goes the other way.
struct LinkIssuer {
    zi::LinkArgs args[2];          // the launch being assembled and the one held back
    zi::LinkFlatArgs flat[2];
    bool is_flat_list = false;     // which of them (expect())
    int32_t n_flat = 0;
    int now = 0;
    bool held = false;
    int dt;
    bool l2;
    hipStream_t stream;
    int64_t launches = 0;

    LinkIssuer(const zi::StepConsts& c, const zi_norm_result* d_norm, uint32_t* h_flag, int dt_, bool l2_, hipStream_t s)
        : dt(dt_), l2(l2_), stream(s)
    {
        for (zi::LinkArgs& a : args) {
            a.n_desc = 0;
            a.n_tiles = 0;
            a.c = c;
            a.d_norm = d_norm;
            a.h_flag = d_norm ? h_flag : nullptr;
        }
    }

    // What the list will be, with addresses as the device sees them, before the first add().
    void expect(const zi_tensor* t, int32_t n_tensors)
    {
        int64_t n = 0, total = 0, longest = 0;
        for (int32_t i = 0; i < n_tensors; ++i) {
            n += t[i].numel > 0;
            total += t[i].numel;
            if (t[i].numel > longest) longest = t[i].numel;
        }
        is_flat_list = n > zi::kMaxLinkDesc && total / n <= StepIssuer::kFlatAverage && longest <= zi::kLinkTilesPerLaunch * zi::kStepTileElems &&
                       is_flat(t, n_tensors, flat[0].list);
        if (!is_flat_list) return;
        flat[0].list.c = args[0].c;
        flat[0].list.d_norm = args[0].d_norm;
        flat[0].h_flag = args[0].h_flag;
        flat[0].n_tiles = 0;
        flat[1] = flat[0];
    }

    // As in StepIssuer, launches are held back by one and those between the first and the last may overlap: the
    // link stays busy while one launch's last tiles return and the next one's first requests are on their way.
    hipError_t issue_held(bool last)
    {
        if (!held) return hipSuccess;
        const bool any_order = !last && launches > 0 && may_overlap(stream);
        ++launches;
        held = false;
        return is_flat_list ? zi::launch_step_link_flat(flat[now ^ 1], dt, l2, any_order, stream)
                            : zi::launch_step_link(args[now ^ 1], dt, l2, any_order, stream);
    }

    hipError_t close()       // the launch being assembled is complete
    {
        if (is_flat_list ? n_flat == 0 : args[now].n_desc == 0) return hipSuccess;
        const hipError_t e = issue_held(false);
        if (is_flat_list) finish_starts(flat[now].list, n_flat);
        now ^= 1;
        held = true;
        args[now].n_desc = 0;
        args[now].n_tiles = 0;
        flat[now].n_tiles = 0;
        n_flat = 0;
        return e;
    }

    hipError_t flush()       // end of the call
    {
        const hipError_t e = close();
        return e != hipSuccess ? e : issue_held(true);
    }

    hipError_t add(float* p, float* m, float* v, const uint16_t* g, uint16_t* p_lp, int64_t numel)
    {
        if (is_flat_list && numel > 0) {
            const int64_t at_most = (numel + zi::kStepTileElems - 1) / zi::kStepTileElems;
            if (n_flat == zi::FlatArgs::kMax || flat[now].n_tiles + at_most > zi::kLinkTilesPerLaunch)
                if (const hipError_t e = close(); e != hipSuccess) return e;
            zi::LinkFlatArgs& a = flat[now];
            a.n_tiles += add_flat(a.list, n_flat++, a.n_tiles, p, choose_head(p, m, v, g, p_lp), numel);
            return hipSuccess;
        }
        while (numel > 0) {
            if (args[now].n_desc == zi::kMaxLinkDesc || args[now].n_tiles >= zi::kLinkTilesPerLaunch) {
                const hipError_t e = close();
                if (e != hipSuccess) return e;
            }
            zi::LinkArgs& a = args[now];
            const int h = choose_head(p, m, v, g, p_lp);
            zi::StepDesc d{};
            d.head = (int32_t)(h < numel ? h : numel);
            const int64_t room = (int64_t)(zi::kLinkTilesPerLaunch - a.n_tiles) * zi::kStepTileElems;
            const int64_t n = numel - d.head <= room ? numel : d.head + room;
            d.p_body = p + d.head; d.m_body = m + d.head; d.v_body = v + d.head; d.g_body = g + d.head;
            d.lp_body = p_lp ? p_lp + d.head : nullptr;
            d.numel = n;
            d.nquad = (n - d.head) / zi::kQuad;
            const int64_t nt = (d.nquad + zi::kStepTileQuads - 1) / zi::kStepTileQuads;
            d.n_tiles = nt < 1 ? 1u : (uint32_t)nt;
            d.first_tile = a.n_tiles;
            a.t[a.n_desc++] = d;
            a.n_tiles += d.n_tiles;
            p += n; m += n; v += n; g += n;
            if (p_lp) p_lp += n;
            numel -= n;
        }
        return hipSuccess;
    }
};

inline zi_status check_norm_args(const zi_tensor* t, int32_t n_tensors, int dt, float loss_scale, zi_norm_result* d_out,
                          void* d_workspace, size_t workspace_bytes)
{
    if (zi_status st = check_dtype(dt)) return st;
    if (zi_status st = check_grad_list(t, n_tensors, loss_scale)) return st;
    if (!d_out) return fail(ZI_ERR_INVALID_ARG, "d_out is NULL");
    if (!aligned(d_out, 8)) return fail(ZI_ERR_ALIGNMENT, "d_out must be 8-byte aligned");
    if (!d_workspace) return fail(ZI_ERR_INVALID_ARG, "d_workspace is NULL");
    if (!aligned(d_workspace, 16)) return fail(ZI_ERR_ALIGNMENT, "d_workspace must be 16-byte aligned");
    if (workspace_bytes < (size_t)zi::kMaxPartials * sizeof(zi::NormPartial))
        return fail(ZI_ERR_INVALID_ARG, "workspace too small: %zu < %zu", workspace_bytes,
                    (size_t)zi::kMaxPartials * sizeof(zi::NormPartial));
    return ZI_OK;
}

// What tells the partials of one launch from anything else that the workspace may hold: a number of 62 bits that the
// process has not used before, from a start that other processes do not share.
inline uint64_t next_norm_number()
{
    static std::atomic<uint64_t> next{(uint64_t)std::chrono::system_clock::now().time_since_epoch().count()};
    return next.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B97F4A7C15ull;      // an odd factor: one to one
}

// Issues the gradient reduction over a list of gradient arrays that the device can reach: partial-sum
// launches of up to NormArgs::kMax tensors, the last of which also makes the final sum.  Whenever the workspace's partial slots
// run out, and at the end of a captured call, a finalize pass folds them; after the first final sum the later ones add to the
// result already in d_out.
struct NormIssuer {
    zi::NormArgs a;
    int32_t n_desc = 0;
    const uint16_t* g0 = nullptr;        // the first of them
    uint32_t n0 = 0;
    zi::NormPartial* partials;
    uint32_t groups = zi::kNormGroups;   // workgroups of a launch, at most
    uint32_t used = 0;                   // partials written since the last finalize
    bool keep = false;                   // see kNormKeepElems
    int64_t tile = zi::kNormTileElems;   // elements of a tile: all launches' (see kNormShortElems)
    int launches = 0;                    // kernels so far
    int finalized = 0;
    int dt;
    float loss_scale;
    zi_norm_result* d_out;
    hipStream_t s;

    NormIssuer(zi::NormPartial* partials_, int dt_, float ls, zi_norm_result* out, hipStream_t st)
        : partials(partials_), dt(dt_), loss_scale(ls), d_out(out), s(st)
    {
        a.n_tiles = 0;
    }
    // What the list will be, before the first add(): gradients in device memory, `total` elements.
    void expect(int64_t total, int64_t n_tensors)
    {
        keep = total <= zi::kNormKeepElems;
        if (total > zi::kNormTileElems && total <= zi::kNormShortElems && n_tensors <= zi::NormArgs::kMax) tile = zi::kNormShortVecs * zi::kVec;
    }
    static int64_t tiles_for(const uint16_t* g, int64_t n, int64_t tile = zi::kNormTileElems)
    {
        const int64_t lead = (int64_t)(-(reinterpret_cast<uintptr_t>(g) / 2) % zi::kVec);
        const int64_t body = n > lead ? (n - lead) / zi::kVec * zi::kVec : 0;
        const int64_t nt = (body + tile - 1) / tile;
        return nt < 1 ? 1 : nt;              // the first tile also owns the unaligned ends
    }
    template <typename Args>
    static void finish_list(Args& a, int32_t n, uint32_t n_tiles)
    {
        a.first_tile[n] = n_tiles;
        for (int32_t i = n + 1; i <= Args::kMax; ++i) a.first_tile[i] = 0xFFFFFFFFu;
        for (int32_t i = 0; i < Args::kGroups; ++i)
            a.group_start[i] = i * Args::kGroup < n ? a.first_tile[i * Args::kGroup] : 0xFFFFFFFFu;
    }
    // final: the launch also makes the final sum.
    hipError_t flush_launch(bool final = false)
    {
        if (n_desc == 0) return hipSuccess;
        hipError_t e = hipSuccess;
        const uint32_t blocks = a.n_tiles < groups ? a.n_tiles : groups;
        if (used + blocks > zi::kMaxPartials && (e = flush_partials()) != hipSuccess) return e;
        a.partials = partials + used;
        const uint64_t number = next_norm_number();
        a.mark_low = (uint32_t)number << 1 | 1u;
        a.mark_high = (uint32_t)(number >> 31) << 1 | 1u;
        a.patience = zi::kNormPatience;
        a.out = final ? d_out : nullptr;
        a.loss_scale = loss_scale;
        a.accumulate = finalized;
        a.n_groups = blocks;
        a.n_before = final ? used : 0;
        const bool is_short = tile != zi::kNormTileElems;
        if (final && n_desc == 1 && used == 0) {
            const zi::NormOne one = {g0, a.partials, a.out, n0, a.n_tiles, blocks, a.mark_low, a.mark_high, a.patience,
                                     loss_scale, a.accumulate};
            e = is_short ? zi::launch_norm_short(one, dt, s) : zi::launch_norm_one(one, dt, keep, s);
        } else if (final && keep && n_desc <= zi::NormFew::kMax && used == 0) {
            zi::NormFew few;
            for (int32_t i = 0; i < n_desc; ++i) {
                few.where[i] = a.where[i];
                few.first_tile[i] = a.first_tile[i];
            }
            finish_list(few, n_desc, a.n_tiles);
            few.n_tiles = a.n_tiles; few.n_groups = a.n_groups;
            few.mark_low = a.mark_low; few.mark_high = a.mark_high; few.patience = a.patience;
            few.loss_scale = a.loss_scale; few.partials = a.partials; few.out = a.out;
            few.n_before = a.n_before; few.accumulate = a.accumulate;
            e = is_short ? zi::launch_norm_short(few, dt, s) : zi::launch_norm_few(few, dt, s);
        } else {
            finish_list(a, n_desc, a.n_tiles);
            // Between two final sums the launches leave partials side by side and may overlap; the first of them and the
            // one with the final sum are ordinary launches (the same order as in StepIssuer).  (A short list is one launch.)
            const bool any_order = used > 0 && !final && may_overlap(s);
            e = is_short ? zi::launch_norm_short(a, dt, s) : zi::launch_norm_partials(a, blocks, dt, keep, any_order, s);
        }
        ++launches;
        used = final ? 0 : used + blocks;
        if (final) finalized = 1;
        n_desc = 0;
        a.n_tiles = 0;
        return e;
    }
    hipError_t flush_partials()
    {
        const hipError_t e = zi::launch_norm_finalize(partials, used, loss_scale, finalized, d_out, s);
        ++launches;
        finalized = 1;
        used = 0;
        return e;
    }
    hipError_t add(const uint16_t* g, int64_t n)
    {
        for (; n > 0; g += zi::kNormMaxPiece, n -= zi::kNormMaxPiece) {
            if (n_desc == zi::NormArgs::kMax)
                if (const hipError_t e = flush_launch(); e != hipSuccess) return e;
            const int64_t m = n < zi::kNormMaxPiece ? n : zi::kNormMaxPiece, tiles = tiles_for(g, m, tile);
            const uint64_t address = reinterpret_cast<uintptr_t>(g);
            if (address >> 48) return hipErrorInvalidValue;
            if (n_desc == 0) {
                g0 = g;
                n0 = (uint32_t)m;
            }
            a.where[n_desc] = address | (uint64_t)(tiles * tile + zi::kNormTileSlack - m) << 48;
            a.first_tile[n_desc++] = a.n_tiles;
            a.n_tiles += (uint32_t)tiles;
        }
        return hipSuccess;
    }
    // Under capture nothing waits for partials by their marks: the marks are the same at every replay, and a workgroup that the
    // last one has given up on leaves its partial with them for the next replay.  Both ways add in one order.  Replays take 1.2 to
    // 1.9 us more so (6.6e4 elements 3.5 -> 4.7, 1.7e7 5.4 -> 7.3, 3.0e8 89.7 -> 91), but for lists that are one workgroup's, where
    // nobody waits (1003 elements 2.4).
    hipError_t finish()
    {
        const bool alone = used == 0 && a.n_tiles == 1;
        if (n_desc > 0 && (alone || !is_captured(s))) return flush_launch(true);
        const hipError_t e = flush_launch();
        return e != hipSuccess ? e : flush_partials();
    }
};

}  // namespace host
}  // namespace zi
