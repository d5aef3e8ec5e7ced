// Internal interface between the C-ABI layer (host) and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "zi.h"
#include "zi_checks.h"

namespace zi {

constexpr int kVec = 8;              // elements per 16-byte vector of a 2-byte array (norm pass)
// Fused step: a lane owns quads of 4 consecutive elements = one 16-byte vector of each fp32 array and
// one 8-byte vector of each 2-byte array, so every wavefront-wide access is one contiguous run.
constexpr int kQuad = 4;
constexpr int kStepThreads = 64;     // one wavefront per workgroup
constexpr int kStepUnroll = 2;       // quads per thread per tile
constexpr int kStepTileQuads = kStepThreads * kStepUnroll;
constexpr int64_t kStepTileElems = (int64_t)kStepTileQuads * kQuad;   // 512 elements per tile
constexpr int kMaxStepDesc = 32;     // tensors (or segments) per fused-step launch
// Workgroup ids are dealt round-robin to the 8 XCDs.  Tiles are renumbered so that, inside every run
// of 8 * kStepXcdRun tiles, each XCD owns kStepXcdRun consecutive tiles (256 KiB of each fp32 array)
// instead of every eighth one: measured +4% on top of the residency cap.
constexpr int kXcds = 8;
#ifndef ZI_STEP_XCD_RUN
#define ZI_STEP_XCD_RUN 128
#endif
constexpr int64_t kStepXcdRun = ZI_STEP_XCD_RUN;

// Dynamic LDS requested (never touched) by the fused step caps its residency, in single-wavefront workgroups per compute unit: on this 1:1 read/write
// stream few, short-lived wavefronts are faster than full occupancy.  LDS is handed out in units of 1280 bytes, 128 on a compute unit (found by
// counting the workgroups that were resident at once; the runtime's occupancy query says one or two more).
constexpr unsigned step_lds(int workgroups) { return (unsigned)(128 / workgroups) * 1280; }

// Half a tile, one quad a lane (adamw_fine_kernel, adamw_fine_list_kernel): twice as many wavefronts with half as many loads each, which live less than
// half as long, so that requests are spread more evenly over time and a launch's last round is shorter.  Step alone, whole / fine tiles, over several
// placements of the arrays: one tensor of 3.0e8 elements 1312..1367 / 1282..1301 us, 64 of 2e7 6104..6178 / 5623..5689.
// Which kernel a launch takes follows from its tiles: fine ones up to kFineShortTiles, where all of its workgroups are resident at once with some places
// to spare (9.5e5 elements at a pace 5.9..6.5, fine 5.4..6.0); from there on paced_quads(), as long as those are (2^20 6.0..6.2 / 6.5..6.9); beyond, fine
// ones again (4.0e6 20.4 / 20.1).
constexpr int kFineTileQuads = kStepThreads;
constexpr uint32_t kFineShortTiles = 7u << 8;      // 9.2e5 elements
constexpr uint32_t kOneRoundTiles = 1u << 12;      // 2.1e6 elements: 16 workgroups on every compute unit
constexpr uint32_t kFineMostTiles = 1u << 25;      // 1.7e10 elements: a launch has less than 2^32 lanes
// One tensor's runs of kFineXcdRun fine tiles go to one XCD each in launches of up to kFineRunTiles; longer ones, and lists, are dealt out as they
// come: then all eight XCDs walk the same few MiB of every array, and it matters little how the arrays lie to each other.  In runs / in none, 1.2e7
// 53.9..54.1 / 54.0..54.9, 3.0e8 1342..1378 / 1282..1301.
constexpr int64_t kFineXcdRun = 1024;
constexpr uint32_t kFineRunTiles = 1u << 15;       // 1.7e7 elements
// Lists whose tensors are arrays of their own go in runs all the same: allocators put such arrays of some MB at the same place of their
// pages, and in plain order all wavefronts then meet on the same channels.  Of views of common buffers the order hardly matters or plain is
// better.  Plain / in runs of 512, own arrays, 21 of 4.0e6 416 / 383, 60 of 4.0e6 1151 / 1096, 15 of 2.0e7 1356 / 1355; views, 60 of 4.0e6 1033 / 1043.
constexpr int64_t kFineListRun = 512;
// Without copies, middling launches of lists stay with whole tiles, and flat ones from kFineListTiles on.  Whole / fine, any lists: 1.3e7 55.1 / 55.4, 2.5e7
// 103.6 / 107.6, 7.6e7 308 / 304; flat ones: 3.0e7 134 / 130, 7.7e7 315 / 321.
constexpr uint32_t kBareListTiles = 1u << 15, kBareListMostTiles = 3u << 15;       // 1.7e7 to 5.0e7 elements
constexpr uint32_t kFineListTiles = 1u << 16;      // 3.4e7 elements
// And many tensors of few tiles each do, whose second halves are often empty: 203 tensors with 1.0e5 elements 13.1 / 13.7, 998 with 1.2e6 30.3 / 31.1; but
// 118 with 6.0e5 7.2 / 6.4.
constexpr uint32_t kManyTensors = 64, kFewTiles = 9;
// Quads that the first fine tile of a body at this address is short of, and the fine tiles of a body.
__host__ __device__ inline uint32_t fine_shift(uintptr_t p_body) { return (uint32_t)(p_body / 16) % kFineTileQuads; }
__host__ __device__ inline uint32_t fine_count(uint32_t nquad, uint32_t shift)
{
    return (uint32_t)(((uint64_t)nquad + shift + kFineTileQuads - 1) / kFineTileQuads);
}
enum class Steps { kOne, kList, kFlat };
inline bool fine_tiles(uint32_t n_tiles, Steps kind, bool copies, uint32_t n_tensors)     // of lists, where paced_quads() says 0
{
    if (n_tensors > kManyTensors && n_tiles < kFewTiles * n_tensors) return false;
    if (kind == Steps::kList && !copies && n_tiles > kBareListTiles && n_tiles <= kBareListMostTiles) return false;
    if (kind == Steps::kFlat && !copies && n_tiles > kFineListTiles) return false;
    return n_tiles <= kFineShortTiles || (n_tiles > kOneRoundTiles && n_tiles < kFineMostTiles);
}
// Launches whose workgroups are all resident at once (16 on a compute unit), at a measured pace (adamw_paced_kernel, adamw_paced_list_kernel): quads that
// a lane takes, 0: not so.  Step alone, all loads up front / at a pace, two quads 1.8e6 10.5 / 9.1, three (fine tiles / at a pace) 3.0e6 15.9 / 14.7,
// four 3.6e6 18.8 / 17.4; four stop paying at 14 on a compute unit.  Lists have tables of whole tiles, which are two quads: 12 tensors of 2.0e6 12.8 /
// 11.5; with 20, 24 or 32 workgroups on a compute unit for longer ones they are no faster than fine tiles.
// Stores are paced too in launches of more than so many workgroups: loads only / both, one tensor 1.95e6 9.8 / 9.9, 2.0e6 10.9 / 10.5; lists 1.4e6
// 9.3 / 9.2, 2.0e6 12.0 / 11.5.
constexpr uint32_t kMostPacedTiles = 7u << 10;     // 3.7e6 elements
constexpr uint32_t kPacedStoresOne = 15u << 8, kPacedStoresList = 11u << 8;
constexpr int kMostPaced = 4;
inline int paced_quads(uint32_t n_tiles, Steps kind)
{
    if (n_tiles <= kFineShortTiles || n_tiles > (kind == Steps::kOne ? kMostPacedTiles : kOneRoundTiles)) return 0;
    constexpr uint32_t per_quad = kOneRoundTiles / kStepUnroll;
    return n_tiles <= kOneRoundTiles ? kStepUnroll : (int)((n_tiles + per_quad - 1) / per_quad);
}
// Resident workgroups per compute unit: what counts is how many have loads in flight at a time.  Without a copy to write they live shorter, and
// lists wait for the lookup in front of their loads.  us by 9 / 10 / 11 / 12 / 14 / 16 / 18 / 21: one tensor of 1.2e7 53.9 / 53.8 / 53.3 / 53.4 / 52.9 /
// 53.3 / 54.1 / 54.5, of 3.0e8 1272 / 1254 / 1260 / 1272 / 1278 / 1300 / 1317 / 1339; 72 of 4.2e6 1286 / 1275 / 1270 / 1266 / 1272 / 1289 / 1302 / 1330; 200
// flat ones of 2e4 22.5 / 21.7 / 21.3 / 21.2 / 20.7 / 20.1 / 19.9 / 20.0.
constexpr unsigned kPacedLds = step_lds(16);
inline unsigned fine_lds(uint32_t n_tiles, Steps kind, bool copies, bool norm)
{
    const bool waits = norm && !copies;
    if (kind == Steps::kOne) return step_lds(n_tiles <= kFineRunTiles ? 16 : waits ? 14 : 11);
    if (n_tiles <= kFineListTiles) return step_lds(kind == Steps::kFlat ? 18 : 16);
    return step_lds(waits ? 16 : 14);
}
inline unsigned whole_tiles_lds(uint32_t n_tiles) { return step_lds(n_tiles <= kOneRoundTiles ? 16 : 7); }

// A tile of the reduction is 16,384 elements, one round of loads for a workgroup.  Gradients that are to stay in the
// memory-side cache (kNormKeepElems) are read by 512 threads with four vectors each, longer lists by 256 with eight: in
// us, 512 / 256 threads, 6.6e4 elements 2.95 / 3.19, 1.0e6 3.47 / 3.68, 4.2e6 3.48 / 3.68, 3.1e8 91.9 / 91.4, 1.3e9 374 / 370.
constexpr int kNormTileVecs = 2048;
constexpr int kNormKeepThreads = 512, kNormStreamThreads = 256;
constexpr int64_t kNormTileElems = (int64_t)kNormTileVecs * kVec;   // 16384 elements per workgroup iteration
// Short lists, of more than one tile and up to kNormShortElems elements, in tiles of one vector a thread (short_sumsq_partial_kernel): four times as many
// compute units have a share of the loads and of the conversions.  Tiles of 16,384 / 8192 / 4096 elements, 512 threads, us: 1.6e4 2.44 / 2.67 / 2.57,
// 6.6e4 3.30 / 2.88 / 2.78, 3.0e5 3.08 / 3.50 / 2.92, 6.0e5 3.67 / 3.02 / 2.89, 1.0e6 3.59 / 3.38 / 3.36, 1.5e6 3.25 / 3.38 / 3.70, 2.1e6
// 3.57 / 3.44 / 3.66, 4.2e6 4.41 / 4.37 / 4.59; 24 tensors with 1.2e5 4.25 / 4.11 / 3.94, 100 with 1.5e5 4.31 / 4.02 / 3.94, 32 with 9.4e5 3.91 / 3.78 /
// 3.61, 200 with 4.0e6 5.70 / 5.75 / 6.64.  (256 threads 0.1 to 0.3 more, 128 up to 1.)
constexpr int kNormShortVecs = 512;
constexpr int64_t kNormShortElems = (int64_t)1 << 20;
// Workgroups of a partial-sum launch (two per compute unit, 64 KiB of loads in flight in each).  Microseconds
// for partials and final sum together on 2.5e7 / 3.0e8 / 1.3e9 elements and on a list of 288 tensors with 3.0e8:
// 512: 12.0 / 91 / 372 / 99, 1024: 11.8 / 92 / 379 / 106, 2048: 11.8 / 92 / 376 / 105, 4096: 11.5 / 94 / 379 / 109;
// a contiguous run of tiles per workgroup 12.2 / 94 / 378 / 101, half the loads in flight 13.0 / 92 / 376 / 100,
// single-wavefront workgroups 12.7 / 92 / 373 / 105 at best.
constexpr int kNormGroups = 512;
// Calls of up to this many elements (176 of the 256 MiB of the memory-side cache) read the gradients with ordinary
// loads, which leave them there for the step that reads them next; streaming loads pass the cache by.  In us, streaming / ordinary:
//   elements                                      1.6e7        3.4e7        6.7e7        9.2e7
//   norm and step, one call after the other       83.2 / 81.5  168 / 160    318 / 300    443 / 413
//     a kernel has just written the gradients     84.2 / 80.3  168 / 160    318 / 303    437 / 417
//     the cache is full of what a kernel has just written elsewhere
//                                                 84.3 / 86.2  168 / 172    320 / 326    441 / 448
//   norm alone, cold but clean                    10.6 / 10.7  16.1 / 16.0  24.7 / 25.7  31.9 / 33.4
//     a kernel has just written the gradients     10.8 / 9.8   15.3 / 14.7  23.5 / 23.1  30.8 / 32.0
//     the cache is full of what a kernel has just written elsewhere
//                                                 10.5 / 16.3  15.8 / 28.6  24.4 / 50.9  31.8 / 69.0
// What a kernel has written elsewhere leaves the cache during the reduction then, 38 us for all of it, of which the step gives
// back most.  The first 176 MiB of longer calls, read last and so, would gain a step the same 24 us (1.0e8 elements 470 / 447, 2.6e8
// 1219 / 1197), but with the cache full of other data both together lose 11 to 16 us (471 / 482, 1219 / 1235), and the reduction
// alone takes 34.1 / 71.7 and 79.8 / 118 us: those calls stream as a whole.
constexpr int64_t kNormKeepElems = (int64_t)11 << 23;
// Gradients in host memory are bound by the link, which few requests in flight fill: GB/s by workgroups
// 32: 55.9, 64: 57.5, 128: 57.4, 256: 56.4, 1024: 55.9.
constexpr int kNormLinkGroups = 64;
constexpr int64_t kNormMaxPiece = (int64_t)1 << 31;   // longer tensors take several descriptors
constexpr uint32_t kMaxPartials = 16384;   // per-block partial results the workspace holds

// One workgroup's partial sum (device workspace element): the two halves of a double, each in the upper half of a word
// whose lower half is the launch's mark (NormArgs).  A word is written and read as one, so a mark that is there says that
// its half of the sum is too.
struct NormPartial {
    uint64_t low, high;
};

// How often the last workgroup of a reduction looks for the other workgroups' partials before it does their work itself
// (every look is a round trip to memory: about a second).
constexpr uint32_t kNormPatience = 1u << 20;

// One tensor (or one segment of one) as the fused step sees it.  All pointers are device memory.
// The first `head` elements are handled one by one; the 4-element lane vectors (the body) start
// after them (the host picks `head` so that as much of the traffic as possible starts on a 128-byte
// line).  Everything a workgroup would otherwise derive from numel and head is worked out once on
// the host: a wavefront lives for a few microseconds, and every scalar instruction in front of its
// first load is time with nothing in flight.
struct StepDesc {
    float* p_body;         // p + head
    float* m_body;
    float* v_body;
    const uint16_t* g_body;
    uint16_t* lp_body;     // p_lp + head, null if there is no copy
    int64_t numel;
    int64_t nquad;         // whole quads of the body: (numel - head) / 4
    int32_t head;          // 0..63
    uint32_t first_tile;   // index of this tensor's first tile within the launch
    uint32_t n_tiles;      // tiles of this tensor: max(1, ceil(nquad / kStepTileQuads))
    uint32_t reserved;
};

// A launch as it is assembled: launch_step_wide hands it on in the form that its kernel takes.
struct StepArgs {
    StepDesc t[kMaxStepDesc];
    int32_t n_desc;
    StepConsts c;
    const zi_norm_result* d_norm;   // device, may be null
    // first_tile of every descriptor once more, packed, 0xFFFFFFFF beyond n_desc (see ListArgs)
    uint32_t first_tile[kMaxStepDesc];
};

// One tensor (adamw_fine_kernel, adamw_paced_kernel), in few bytes: a call on a short one takes the host longer than the GPU, and what the runtime takes
// for a launch depends on the size of its arguments.  Issue of an empty kernel in us (the runtime runs in one of two modes for
// the life of a process): up to 112 bytes 2.4 or 2.8, 120 to 1024 bytes 2.5 or 3.5 to 3.7, StepArgs' 2.5 KB 2.55 or 3.75, 3.6 KB and
// more 2.55 or 3.8 to 4.1.
struct StepOne {
    float* p_body;         // p + head
    float* m_body;
    float* v_body;
    const uint16_t* g_body;
    uint16_t* lp_body;     // p_lp + head, null if there is no copy
    const zi_norm_result* d_norm;
    double inv_loss_scale;
    uint32_t nquad;
    uint8_t head, tail, scale_is_pow2, max_norm_is_pow2;
    float beta1, beta2, omb1, omb2, eps, step_size, inv_sqrt_bc2;
    float decay;           // of AdamW, or the weight decay of Adam with L2
    float loss_scale, max_grad_norm, host_gscale;
};
static_assert(sizeof(StepOne) <= 112, "kernel arguments");
inline void set_scalars(StepOne& a, const StepConsts& c, bool l2, const zi_norm_result* d_norm)
{
    a.d_norm = d_norm;
    a.inv_loss_scale = c.inv_loss_scale;
    a.scale_is_pow2 = (uint8_t)c.scale_is_pow2;
    a.max_norm_is_pow2 = (uint8_t)c.max_norm_is_pow2;
    a.beta1 = c.beta1; a.beta2 = c.beta2; a.omb1 = c.omb1; a.omb2 = c.omb2;
    a.eps = c.eps; a.step_size = c.step_size; a.inv_sqrt_bc2 = c.inv_sqrt_bc2;
    a.decay = l2 ? c.weight_decay : c.decay;
    a.loss_scale = c.loss_scale; a.max_grad_norm = c.max_grad_norm; a.host_gscale = c.host_gscale;
}

// Launches over many tensors (adamw_list_kernel, adamw_fine_list_kernel, adamw_paced_list_kernel), which a workgroup looks up in groups.  A list whose tensors are
// views at the same places of five flat buffers, as the partitions of a sharded optimizer are, needs one place per
// tensor (FlatArgs); any other list five addresses (ListArgs).
struct ListDesc {
    float* p_body;         // p + head
    float* m_body;
    float* v_body;
    const uint16_t* g_body;
    uint16_t* lp_body;     // p_lp + head, null if there is no copy
    uint32_t nquad;
    uint16_t head, tail;   // elements in front of the quads (0..63) and behind them (0..3)
};

struct ListArgs {
    static constexpr int kGroup = 8, kGroups = 8, kMax = kGroup * kGroups;
    ListDesc t[kMax];
    uint32_t first_tile[kMax];              // 0xFFFFFFFF beyond the list
    uint32_t group_start[kGroups];          // first_tile of every group's first
    StepConsts c;
    const zi_norm_result* d_norm;
};
static_assert(sizeof(ListArgs) < 4096, "kernel arguments");
constexpr int kMaxListDesc = ListArgs::kMax;

struct FlatDesc {
    uint32_t body;         // elements from the list's first tensor to this one's body
    uint32_t nquad;
};

template <int GROUPS>
struct FlatList {
    static constexpr int kGroup = 16, kGroups = GROUPS, kMax = kGroup * kGroups;
    FlatDesc t[kMax];
    uint32_t first_tile[kMax];
    uint32_t group_start[kGroups];
    float *p, *m, *v;      // the list's first tensor
    const uint16_t* g;
    uint16_t* lp;          // null if there are no copies
    StepConsts c;
    const zi_norm_result* d_norm;
    uint8_t head[kMax], tail[kMax];
};
struct FlatArgs : FlatList<16> {};
static_assert(sizeof(FlatArgs) < 4096, "kernel arguments");
// Up to 32 tensors with kFewElems elements or less in all, which take the host longer than the GPU: 568 bytes instead of
// StepArgs' 2.5 KB, and no StepIssuer (StepOne says what that is worth).  Norm and step together, StepArgs and NormArgs / FlatFew and
// NormFew, us: issue without the binding, 2 tensors 9.5 / 8.9, 16 9.8 / 9.3, 32 10.1 / 9.8; on the GPU 24 tensors of 1.0e4
// elements 8.1 / 7.6, 12 of 8.0e4 9.8 / 9.6, 32 of 3.0e4 10.6 / 10.3, 24 with 1.6e6 13.0 / 12.6, 23 with 1.7e6 14.2 / 14.2,
// 24 of 1.0e5 17.0 / 17.2.
struct FlatFew : FlatList<2> {};
constexpr int64_t kFewElems = (int64_t)1 << 21;

// The step over state in page-locked host memory (adamw_link_kernel): a persistent grid of
// single-wavefront workgroups that read and write the host arrays over the link themselves.
// The kernel is bound by the link's two directions, so the grid only has to keep the link's queues full.
// Measured on three pinned arrays updated in place, GB/s per direction by workgroups, two hosts:
// 32: 47.0 / 49.2, 64: 50.1 / 46.5, 96: 49.4 / 49.5, 128: 48.8 / 49.6, 256: 45.2, 512: 44.4.  96 is within 2%
// of the best on both.  Four quads a lane, one quad a lane, larger workgroups and loads of the next tile
// in front of this one's stores moved it by 1% up or down.
constexpr int kLinkGroups = 96;
constexpr int kMaxLinkDesc = 48;                       // segments per launch (the argument block stays below 4 KiB)
constexpr uint32_t kLinkTilesPerLaunch = 1u << 19;     // 2^28 elements, some 65 ms of link time

struct LinkArgs {
    StepDesc t[kMaxLinkDesc];       // addresses as the device sees them
    int32_t n_desc;
    uint32_t n_tiles;
    StepConsts c;
    const zi_norm_result* d_norm;   // device, may be null
    uint32_t* h_flag;               // page-locked: receives d_norm->found_inf; null without d_norm
};
static_assert(sizeof(LinkArgs) < 4096, "kernel arguments");

// The same for more short tensors than kMaxLinkDesc at the same places of five flat buffers: 256 of them.  A launch of 48
// tensors of a tile or two leaves half of the workgroups without work, and its round trips over the link are paid per launch.
struct LinkFlatArgs {
    FlatArgs list;                  // addresses as the device sees them
    uint32_t n_tiles;
    uint32_t* h_flag;
};
static_assert(sizeof(LinkFlatArgs) < 4096, "kernel arguments");

// Copies of 2-byte arrays between device and page-locked host memory by a kernel (link_copy_kernel): many segments in
// one launch, in blocks of 2^14 elements that report to the host when they have arrived, or in pieces of 2^12 (one
// round of loads for a wavefront) where nobody waits for a part.
constexpr int64_t kCopyBlockElems = (int64_t)1 << 14;
constexpr int64_t kCopyPieceElems = (int64_t)1 << 12;
constexpr int kMaxCopySegs = 32;
constexpr int kCopyGroups = 96;

struct CopySeg {
    const uint16_t* src;
    uint16_t* dst;
    int64_t elems;
    uint32_t first_tile;   // index of the segment's first block within the launch
    uint32_t flag;         // index of its first block's flag
};

struct CopyArgs {
    CopySeg t[kMaxCopySegs];
    uint32_t n_segs, n_blocks;
    uint32_t* flags;       // page-locked, null: the blocks do not report
    uint32_t serial;       // what a block's flag becomes once the block is at its destination
};

// The reduction over a list: 12 bytes a tensor, so that a launch takes 320 (with address, length and first tile in 16 bytes
// it took 224), which a workgroup looks up in groups as adamw_list_kernel does, in two round trips to the scalar cache where
// halving takes eight.  Reduction alone, us: 288 tensors with 3.0e8 elements 94 -> 90, 300 of 1..20,000 8.7 -> 5.1 (two launches and
// a final sum before), 1000 of 1..100,000 43 -> 29, 200 of 1..40,000 5.1 / 5.2.
template <int GROUPS>
struct NormList {
    static constexpr int kGroup = 16, kGroups = GROUPS, kMax = kGroup * kGroups;
    // Address of the tensor in the lower 48 bits (the GPU has no others); above, how many elements its length is
    // short of its tiles * the elements of a tile + kNormTileSlack.
    uint64_t where[kMax];
    uint32_t first_tile[kMax + 1];  // behind the list: n_tiles, then 0xFFFFFFFF
    uint32_t group_start[kGroups];  // first_tile of every group's first
    uint32_t n_tiles;
    uint32_t n_groups;              // workgroups of the launch
    uint32_t mark_low, mark_high;   // neither is zero; no other launch of the process has the same two
    uint32_t patience;              // kNormPatience
    float loss_scale;
    NormPartial* partials;          // of this launch
    // The last launch of a reduction makes the final sum (null: not this one), over its own partials and the n_before in
    // front of them that launches before it left.
    zi_norm_result* out;
    uint32_t n_before;
    int32_t accumulate;             // adds to what is in *out
};
struct NormArgs : NormList<20> {};
static_assert(sizeof(NormArgs) < 4096, "kernel arguments");
struct NormFew : NormList<2> {};        // short lists of up to 32 tensors, as FlatFew
// Elements that a tensor's first tile takes beside its vectors: at most 7 in front of them and 7 behind.
constexpr uint32_t kNormTileSlack = 2 * (kVec - 1);

// The same for one tensor, small as StepOne is.
struct NormOne {
    const uint16_t* g;
    NormPartial* partials;
    zi_norm_result* out;
    uint32_t numel, n_tiles, n_groups, mark_low, mark_high, patience;
    float loss_scale;
    int32_t accumulate;
    static constexpr uint32_t n_before = 0;
};
static_assert(sizeof(NormOne) <= 112, "kernel arguments");

// Launchers (zi_kernels.hip).  Each returns the hipError_t of the launch.
// any_order: may run beside the launches in front of it on the stream (see StepIssuer for where that is safe).
hipError_t launch_step_wide(const StepArgs& a, uint32_t n_tiles, int dt, bool l2, bool any_order, hipStream_t s);
hipError_t launch_step_one(const StepOne& a, int dt, bool l2, bool any_order, hipStream_t s);
hipError_t launch_step_few(const FlatFew& a, uint32_t n_tiles, int dt, bool l2, hipStream_t s);
hipError_t launch_step_list(const ListArgs& a, uint32_t n_tiles, int dt, bool l2, bool any_order, hipStream_t s);
hipError_t launch_step_flat(const FlatArgs& a, uint32_t n_tiles, int dt, bool l2, bool any_order, hipStream_t s);
hipError_t launch_link_copy(const CopyArgs& a, hipStream_t s);
hipError_t launch_step_link(const LinkArgs& a, int dt, bool l2, bool any_order, hipStream_t s);
hipError_t launch_step_link_flat(const LinkFlatArgs& a, int dt, bool l2, bool any_order, hipStream_t s);
// keep: read with ordinary loads instead of streaming ones (kNormKeepElems).
hipError_t launch_norm_partials(const NormArgs& a, uint32_t n_blocks, int dt, bool keep, bool any_order, hipStream_t s);
hipError_t launch_norm_one(const NormOne& a, int dt, bool keep, hipStream_t s);
hipError_t launch_norm_few(const NormFew& a, int dt, hipStream_t s);      // ordinary loads
hipError_t launch_norm_short(const NormOne& a, int dt, hipStream_t s);    // the same three in tiles of kNormShortVecs
hipError_t launch_norm_short(const NormFew& a, int dt, hipStream_t s);
hipError_t launch_norm_short(const NormArgs& a, int dt, hipStream_t s);
hipError_t launch_norm_finalize(const NormPartial* partials, uint32_t count, float loss_scale, int accumulate,
                                zi_norm_result* d_out, hipStream_t s);

hipError_t launch_norm_refresh(zi_norm_result* d_result, float loss_scale, hipStream_t s);
hipError_t launch_hbm_probe(void* a, void* b, int64_t n4, int mode, float* sink, hipStream_t s);

}  // namespace zi
