// Entry points around the streamed step that move the 2-byte arrays rather than the state:
//   zi_grad_offload / zi_grad_offload_wait / zi_grad_offload_order   freshly produced gradient partitions
//       leave for host memory on the engine's device-to-host stream while their producer keeps running;
//   zi_adamw_step_cpu   the step itself on the host CPUs over host-resident state, with only gradients
//       coming down the link and the low-precision copy going up, the three stages overlapped
//       through the engine's pinned ring.
// See include/zi.h for the contract of every call.
#include <hip/hip_runtime.h>

#include <cerrno>
#include <chrono>
#include <cstring>

#include "zi_engine_internal.h"

using namespace zi::host;

// ============================================================================ gradient offload

// The copy is the runtime's: link_copy_kernel is faster for partitions of 1 to 4 MiB while the GPU is idle, but these
// calls are made beside the backward pass, and there its workgroups keep the producer's waiting.
// Per call of a row of offloads on an idle GPU, us, copy / kernel: 64 KiB 15 / 22, 256 KiB 23 / 22, 1 MiB 69 / 25, 4 MiB
// 206 / 82, 16 MiB 306 / 307.  40 partitions, each behind a matrix product of 110 us, us until the producer is done
// (4380 without offloads) / until the last partition has arrived, copy and kernel:
// 256 KiB 4313 / 4377 and 4374 / 4412, 1 MiB 4427 / 4573 and 4915 / 4966, 4 MiB 4764 / 8284 and 6928 / 7037; each behind a
// kernel of 347 us that streams 2 GiB (13,860 without): 4 MiB 14,020 / 14,134 and 14,903 / 15,011.
extern "C" zi_status zi_grad_offload(zi_engine* e, const void* d_src, void* h_dst, size_t bytes,
                                     void* producer_stream)
{
    if (zi_status st = check_engine(e)) return st;
    if (bytes == 0) return ZI_OK;
    if (!d_src || !h_dst) return fail(ZI_ERR_INVALID_ARG, "d_src and h_dst must not be NULL");
    PointerChecker reach;
    if (memory_kind(d_src) != 0) return fail(ZI_ERR_INVALID_ARG, "d_src must be device memory");
    if (zi_status st = reach.check(d_src, bytes, -1, "d_src")) return st;
    if (memory_kind(h_dst) != 1 || memory_kind(static_cast<const char*>(h_dst) + bytes - 1) != 1)
        return fail(ZI_ERR_INVALID_ARG, "h_dst (%zu bytes) must be page-locked host memory", bytes);
    ZI_HIP(hipSetDevice(e->device));

    // One event per call orders the copy after everything the producer has enqueued so far.  The
    // events are reused round-robin; before a reuse, the copy that waited on the event is long
    // done (64 offloads ago), which the host makes sure of.
    const int idx = (int)(e->n_offloads % kOffloadEvents);
    if (e->n_offloads >= (uint64_t)kOffloadEvents) ZI_HIP(hipEventSynchronize(e->ev_offload[idx]));
    ZI_HIP(hipEventRecord(e->ev_offload[idx], (hipStream_t)producer_stream));
    ZI_HIP(hipStreamWaitEvent(e->s_d2h, e->ev_offload[idx], 0));
    ZI_HIP(hipMemcpyAsync(h_dst, d_src, bytes, hipMemcpyDeviceToHost, e->s_d2h));
    ++e->n_offloads;
    e->offload_pending = true;
    return ZI_OK;
}

extern "C" zi_status zi_grad_offload_wait(zi_engine* e)
{
    if (zi_status st = check_engine(e)) return st;
    if (!e->offload_pending) return ZI_OK;
    ZI_HIP(hipSetDevice(e->device));
    ZI_HIP(wait_for_offloads(e));
    e->offload_pending = false;
    return ZI_OK;
}

extern "C" zi_status zi_grad_offload_order(zi_engine* e, void* consumer_stream)
{
    if (zi_status st = check_engine(e)) return st;
    ZI_HIP(hipSetDevice(e->device));
    ZI_HIP(order_after_offloads(e, (hipStream_t)consumer_stream));
    return ZI_OK;
}

// ====================================================================== the step on the host CPUs

namespace {

// Tasks are blocks of link_copy_kernel: 64 KiB of each fp32 array.  A chunk of 2^24 elements is 1024
// tasks, so the barrier at the end of every chunk finds the threads within one short task of each
// other (2^18-element tasks measured 4% slower, 2^16 2% slower).
constexpr int64_t kCpuBlockElems = zi::kCopyBlockElems;
// Stepped blocks whose copy the calling thread sends up together while the others go on: 2 MiB.
// A use of one segment that is no longer than that goes up when it is stepped, beside the next use, and then the runtime's
// copy is the cheaper way: per call with 16 threads, us, kernel / copy (three runs each), 8.4e6 elements in chunks of
// 1 MiB 1914..1942 / 1728..1846, 1.7e7 in chunks of 2 MiB 3087..3095 / 2830..2956, in chunks of 4 MiB 2466..2608 /
// 2360..2632; 3.4e7 in chunks of 8 MiB 4442..5478 / 5287..5483.  For the last use, whose upload everybody waits for, the
// kernel is: 3.0e4 elements 83..93 / 89..96.
constexpr size_t kUploadBlocks = 64;

// One slot use.  A thread steps a block as soon as the block's gradients have arrived, and the calling thread,
// which works on blocks like the others, sends up what is finished from the front between two of its own: within a
// use the fetch, the step and the upload of different blocks overlap, so a state of one chunk does not wait
// for its whole fetch nor expose its whole upload.
struct CpuJob {
    zi_engine* e;
    const CpuBlock* blocks;
    size_t n_blocks;
    uint32_t serial;
    zi::StepConsts c;
    float gscale;
    int dt;
    bool l2;
    uint32_t* done;               // per block
    size_t sent = 0;              // blocks whose copy is on its way (or in its place)
    hipError_t upload_error = hipSuccess;

    // Sends up the copies of blocks [sent, to), neighbours of one segment as one.
    void upload(size_t to)
    {
        CopyIssuer up(e->s_h2d, nullptr, 0);
        while (sent < to && upload_error == hipSuccess) {
            const CpuBlock& b = blocks[sent];
            int64_t n = b.n;
            size_t next = sent + 1;
            if (b.lp_device)
                while (next < to && blocks[next].lp_device == b.lp_device + n && blocks[next].lp == b.lp + n &&
                       blocks[next].lp_by_copy == b.lp_by_copy)
                    n += blocks[next++].n;
            if (b.lp_device) {
                upload_error = b.lp_by_copy ? hipMemcpyAsync(b.lp_device, b.lp, (size_t)n * 2, hipMemcpyHostToDevice, e->s_h2d)
                                            : up.add(b.lp, b.lp_device, n, 0);
                e->stats.n_copies += b.lp_by_copy;
                e->stats.bytes_h2d += (uint64_t)n * 2;
            }
            sent = next;
        }
        if (upload_error == hipSuccess) upload_error = up.flush();
    }
};

// Waits until a block's gradients are in the ring.  The kernel that brings them ends whatever happens; if its
// stream reports an error, or is done without having raised the flag, the wait ends with an error.
bool wait_arrived(const CpuJob& job, const uint32_t* flag)
{
    for (uint64_t spins = 1; __atomic_load_n(flag, __ATOMIC_ACQUIRE) != job.serial; ++spins) {
        __builtin_ia32_pause();
        if (spins % (1u << 16)) continue;
        const hipError_t e = hipStreamQuery(job.e->s_d2h);
        if (e == hipErrorNotReady) continue;
        return e == hipSuccess && __atomic_load_n(flag, __ATOMIC_ACQUIRE) == job.serial;
    }
    return true;
}

// Brings the norm result to e->h_norm and waits for it, and with it for everything on the stream so far.  A kernel raises a flag behind
// its 32 bytes (the runtime's copy and the wait for its signal took 13.5 us); what it may not touch, or on another device's
// stream, the runtime copies.  The flag says that earlier kernels have ended, and what they wrote in this device's memory is
// there for the kernels to come; written to page-locked memory or to another device it is certain to be there only once the stream has been synchronised,
// and then the runtime's copy in front of that is the quicker one (skipped step 14 us, with the kernel 17).
zi_status read_norm(zi_engine* e, const zi_norm_result* d_norm, hipStream_t user, bool flag_is_enough)
{
    int owner = -1;
    hipDevice_t on = e->device;
    const int kind = memory_kind(d_norm, &owner);
    if (user && hipStreamGetDevice(user, &on) != hipSuccess) on = -1;
    if (on < 0) (void)hipGetLastError();
    HostNorm* const host = reinterpret_cast<HostNorm*>(e->h_norm);
    if (flag_is_enough && kind == 0 && owner == e->device && on == e->device) {
        const uint32_t serial = ++e->norm_serial;
        CopyIssuer out(user, &host->arrived, serial);
        ZI_HIP(out.add((const uint16_t*)d_norm, (uint16_t*)e->h_norm, sizeof(zi_norm_result) / 2, 0));
        ZI_HIP(out.flush());
        for (int spins = 0; spins < (1 << 14); ++spins) {
            if (__atomic_load_n(&host->arrived, __ATOMIC_ACQUIRE) == serial) return ZI_OK;
            __builtin_ia32_pause();
        }
    } else {
        ZI_HIP(hipMemcpyAsync(e->h_norm, d_norm, sizeof(zi_norm_result), hipMemcpyDeviceToHost, user));
    }
    ZI_HIP(hipStreamSynchronize(user));
    return ZI_OK;
}

int run_cpu_block(void* ctx, size_t index, int who)
{
    CpuJob& job = *static_cast<CpuJob*>(ctx);
    const CpuBlock& b = job.blocks[index];
    if (b.arrived && !wait_arrived(job, b.arrived)) return EIO;
    host_step_range(job.c, job.gscale, job.dt, job.l2, b.p, b.m, b.v, b.g, b.lp, 0, b.n);
    __atomic_store_n(&job.done[index], 1u, __ATOMIC_RELEASE);
    if (who == 0) {
        size_t front = job.sent;
        while (front < job.n_blocks && __atomic_load_n(&job.done[front], __ATOMIC_ACQUIRE)) ++front;
        if (front >= job.sent + kUploadBlocks) job.upload(front);
    }
    return 0;
}

}  // namespace

extern "C" zi_status zi_adamw_step_cpu(zi_engine* e, const zi_tensor* t, int32_t n_tensors, zi_lp_dtype dt,
                                       const zi_adamw_config* cfg, const zi_norm_result* d_norm,
                                       int32_t n_threads, void* hip_stream)
{
    ZI_GUARD_BEGIN
    if (zi_status st = check_engine(e)) return st;
    if (!host_step_supported()) return fail(ZI_ERR_UNSUPPORTED, "the host step needs a CPU with AVX2, FMA and F16C");
    if (n_threads < 1 || n_threads > 256) return fail(ZI_ERR_INVALID_ARG, "n_threads must be in 1..256");
    if (zi_status st = check_dtype((int)dt)) return st;
    if (zi_status st = check_config(cfg)) return st;
    if (zi_status st = check_step_tensors(t, n_tensors)) return st;
    if (d_norm && !aligned(d_norm, 8)) return fail(ZI_ERR_ALIGNMENT, "d_norm must be 8-byte aligned");
    if (zi_status st = check_kernel_visible(d_norm, sizeof(zi_norm_result), -1, "d_norm")) return st;
    ZI_HIP(hipSetDevice(e->device));
    hipStream_t user = (hipStream_t)hip_stream;
    e->stats = zi_stream_stats{};
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (user && hipStreamIsCapturing(user, &capture) != hipSuccess) (void)hipGetLastError();
    if (capture != hipStreamCaptureStatusNone) return fail(ZI_ERR_HIP, "the stream is being captured; this call waits for it");

    // p, m, v: host memory of any kind (the CPUs work on them in place).  g, p_lp: device memory
    // (staged through the pinned ring, chunk by chunk) or host memory (used in place).
    bool any_device = false;
    bool all_here = true;         // p, m, v in ordinary memory, g and p_lp on this device: see read_norm
    PointerChecker reach;
    e->src.resize((size_t)n_tensors);
    for (int32_t i = 0; i < n_tensors; ++i) {
        StateSrc& S = e->src[(size_t)i];
        S = StateSrc{};
        S.ptr[0] = (char*)t[i].p; S.ptr[1] = (char*)t[i].m; S.ptr[2] = (char*)t[i].v;
        S.g = t[i].g; S.p_lp = t[i].p_lp; S.numel = t[i].numel;
        S.g_host = S.lp_host = true;
        if (t[i].numel == 0) continue;
        const size_t n = (size_t)t[i].numel;
        for (int w = 0; w < 3; ++w) {
            const int k0 = memory_kind(S.ptr[w]), k1 = memory_kind(S.ptr[w] + n * 4 - 1);
            if (k0 == -2) return fail(ZI_ERR_HIP, "no usable HIP device (pointer query failed)");
            if ((k0 != 1 && k0 != 2) || k1 != k0)
                return fail(ZI_ERR_INVALID_ARG, "tensor %d: p, m, v must be host memory", i);
            all_here = all_here && k0 == 2;
        }
        int owner = e->device;
        const int gk = memory_kind(S.g, &owner);
        if (gk < 0) return fail(ZI_ERR_INVALID_ARG, "tensor %d: g is neither device nor host memory", i);
        all_here = all_here && (gk == 2 || (gk == 0 && owner == e->device));
        if (gk == 0) {
            if (zi_status st = reach.check(S.g, n * 2, i, "g")) return st;
            S.g_host = false;
            S.g_peer = owner != e->device;
            any_device = true;
        }
        if (S.p_lp) {
            const int lk = memory_kind(S.p_lp, &owner);
            if (lk < 0) return fail(ZI_ERR_INVALID_ARG, "tensor %d: p_lp is neither device nor host memory", i);
            all_here = all_here && (lk == 2 || (lk == 0 && owner == e->device));
            if (lk == 0) {
                if (zi_status st = reach.check(S.p_lp, n * 2, i, "p_lp")) return st;
                S.lp_host = false;
                S.lp_peer = owner != e->device;
                any_device = true;
            }
        }
    }
    const int n_h = e->n_hslots;
    if (any_device && n_h < 3)
        return fail(ZI_ERR_INVALID_ARG, "device-resident gradients or copy need a pinned ring of at least 3 slots "
                                        "(ZI_OPT_HOST_RING_SLOTS)");
    if (!e->pool_step || e->pool_step->threads() != n_threads) {
        delete e->pool_step;
        e->pool_step = new TaskPool(n_threads);
    }

    e->plan_numel.resize((size_t)n_tensors);
    for (int32_t i = 0; i < n_tensors; ++i) e->plan_numel[(size_t)i] = t[i].numel;
    int64_t n_uses = 0;
    plan_chunks(e->plan_numel.data(), n_tensors, e->chunk_elems, e->segs, n_uses);
    index_uses(e->segs, n_uses, e->use_begin);
    const std::vector<Segment>& segs = e->segs;
    const std::vector<size_t>& use_begin = e->use_begin;

    // The flag and the sum of squares come to the host first: a skipped step touches, moves and waits for nothing else.
    zi::StepConsts k = make_consts(*cfg);
    float gscale = k.host_gscale;
    if (d_norm) {
        if (zi_status st = read_norm(e, d_norm, user, all_here)) return st;
        if (e->h_norm->found_inf) return ZI_SKIPPED_OVERFLOW;
        gscale = gradient_factor(e->h_norm->sumsq, k);
    }
    // Gradient offloads on their way to host memory are complete before the CPUs read them, and gradients
    // produced on the caller's stream before they are fetched (where the norm is here, that stream has been waited for).
    ZI_HIP(wait_for_offloads(e));
    e->offload_pending = false;
    if (!d_norm) {
        ZI_HIP(hipEventRecord(e->ev_in, user));
        if (any_device) ZI_HIP(hipStreamWaitEvent(e->s_d2h, e->ev_in, 0));
    }

    const auto t0 = std::chrono::steady_clock::now();
    // Around the uses, the host waits for the norm result and for the last upload, and the engine's streams for nothing.  With the runtime's copy of
    // the result, stream waits behind an event for the caller's stream, an event in front of what follows on it, and a wait for the fetches, a
    // call took (us, 16 threads, ordinary state; jobs of few tasks without the whole pool are in that) 1000 elements 110 / 34, 5.0e4 108 / 55,
    // 3.0e5 140 / 102, 1.5e6 315 / 293; page-locked state 115 / 36, 114 / 57, 141 / 101, 297 / 253; from 1.7e7 on no difference beyond that of two
    // runs.  Fetching in front of the flag's way to the host made 1000 elements 57, and a skipped step 40 (one use) to 1290 (two uses of 2^24)
    // where it takes 12.
    // Ring slot u mod n_h carries slot use u: its gradient half is filled by a kernel that reports every block
    // (link_copy_kernel), the CPUs step the use (reading that half, writing the copy half), and the copy half is
    // sent up by the same kind of kernel or by the runtime's copy (kUploadBlocks; arrays of another device).
    // Fetches run `ahead` uses in front of the CPUs; a slot is fetched into again only after the upload of its
    // previous use has left it, which by then is two steps old.
    const int ahead = n_h >= 3 ? n_h - 2 : 1;
    const uint32_t first_serial = e->fill_serial + 1;         // of use 0; use u has first_serial + u
    e->fill_serial += (uint32_t)n_uses;
    auto blocks_of = [](int64_t count) { return (count + kCpuBlockElems - 1) / kCpuBlockElems; };
    auto fetch = [&](int64_t u) -> zi_status {
        const int h = n_h > 0 ? (int)(u % n_h) : 0;
        CopyIssuer in(e->s_d2h, n_h > 0 ? e->fill_flags + (size_t)h * e->flags_per_slot : nullptr, first_serial + (uint32_t)u);
        bool any = false, peer = false;
        uint32_t flag = 0;
        for (size_t j = use_begin[(size_t)u]; j < use_begin[(size_t)u + 1]; ++j) {
            const Segment& sg = segs[j];
            const StateSrc& S = e->src[(size_t)sg.tensor];
            if (!S.g_host) {
                if (!any && u >= n_h) ZI_HIP(hipEventSynchronize(e->ev_back[h]));
                any = true;
                const uint16_t* from = (const uint16_t*)S.g + sg.elem_offset;
                uint16_t* to = e->hslot_g(h) + sg.slot_offset;
                if (S.g_peer) {
                    ZI_HIP(hipMemcpyAsync(to, from, (size_t)sg.count * 2, hipMemcpyDeviceToHost, e->s_d2h));
                    ++e->stats.n_copies;
                    peer = true;
                } else {
                    ZI_HIP(in.add(from, to, sg.count, flag));
                }
                e->stats.bytes_d2h += (size_t)sg.count * 2;
            }
            flag += (uint32_t)blocks_of(sg.count);
        }
        ZI_HIP(in.flush());
        if (peer) ZI_HIP(hipEventRecord(e->ev_fill[h], e->s_d2h));
        return ZI_OK;
    };
    bool uploaded = false;
    auto pipeline = [&]() -> zi_status {
        std::vector<CpuBlock>& blocks = e->cpu_blocks;
        for (int64_t u = 0; u < n_uses && u < ahead; ++u)
            if (zi_status st = fetch(u)) return st;
        // One thread waits for the gradients' producer, and for whoever still reads the copy, not all of them; from here on the caller's
        // stream is no one's to wait for.
        if (!d_norm) ZI_HIP(hipEventSynchronize(e->ev_in));
        for (int64_t u = 0; u < n_uses; ++u) {
            if (u + ahead < n_uses)
                if (zi_status st = fetch(u + ahead)) return st;
            const int h = n_h > 0 ? (int)(u % n_h) : 0;
            const uint32_t* flags = n_h > 0 ? e->fill_flags + (size_t)h * e->flags_per_slot : nullptr;
            blocks.clear();
            bool fetched = false, peer = false, upload = false;
            const bool in_one = use_begin[(size_t)u + 1] - use_begin[(size_t)u] == 1 && u + 1 < n_uses &&
                                blocks_of(segs[use_begin[(size_t)u]].count) <= (int64_t)kUploadBlocks;
            for (size_t j = use_begin[(size_t)u]; j < use_begin[(size_t)u + 1]; ++j) {
                const Segment& sg = segs[j];
                const StateSrc& S = e->src[(size_t)sg.tensor];
                const bool up = S.p_lp && !S.lp_host;
                fetched = fetched || !S.g_host;
                peer = peer || S.g_peer;
                upload = upload || up;
                const uint16_t* g = S.g_host ? (const uint16_t*)S.g + sg.elem_offset : e->hslot_g(h) + sg.slot_offset;
                uint16_t* lp = !S.p_lp ? nullptr
                               : S.lp_host ? (uint16_t*)S.p_lp + sg.elem_offset : e->hslot_lp(h) + sg.slot_offset;
                for (int64_t o = 0; o < sg.count; o += kCpuBlockElems) {
                    const int64_t nb = sg.count - o < kCpuBlockElems ? sg.count - o : kCpuBlockElems;
                    const int64_t at = sg.elem_offset + o;
                    blocks.push_back({(float*)S.ptr[0] + at, (float*)S.ptr[1] + at, (float*)S.ptr[2] + at, g + o,
                                      lp ? lp + o : nullptr, nb, S.g_host || S.g_peer ? nullptr : flags + blocks.size(),
                                      up ? (uint16_t*)S.p_lp + at : nullptr, S.lp_peer || in_one});
                }
            }
            // A ring slot whose upload of `n_h` uses ago is still leaving must not be written yet
            // (uses with host-resident gradients skip the fetch that would have waited for it).
            if (upload && !fetched && u >= n_h) ZI_HIP(hipEventSynchronize(e->ev_back[h]));
            if (peer) ZI_HIP(hipEventSynchronize(e->ev_fill[h]));      // the runtime's copies raise no flags
            e->cpu_done.assign(blocks.size(), 0);
            CpuJob job{e, blocks.data(), blocks.size(), first_serial + (uint32_t)u, k, gscale, (int)dt,
                       cfg->mode == ZI_MODE_ADAM_L2, e->cpu_done.data()};
            if (e->pool_step->run(blocks.size(), run_cpu_block, &job) != 0)
                return fail(ZI_ERR_HIP, "gradients did not arrive in the pinned ring");
            job.upload(blocks.size());
            ZI_HIP(job.upload_error);
            uploaded = uploaded || upload;
            if ((upload || fetched) && u + n_h < n_uses) ZI_HIP(hipEventRecord(e->ev_back[h], e->s_h2d));
            ++e->stats.n_slot_uses;
        }
        // The copy is complete on return.  (The fetches are: every block's flag has been seen.)
        if (uploaded) ZI_HIP(hipStreamSynchronize(e->s_h2d));
        return ZI_OK;
    };
    const zi_status st = pipeline();
    if (st != ZI_OK) drain_streams(e);
    e->stats.seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return st;
    ZI_GUARD_END
}
