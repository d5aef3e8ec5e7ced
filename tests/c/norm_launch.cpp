// One launch of the reduction's kernel with a patience of the test's choice, through the library's own launcher.
#define __HIP_PLATFORM_AMD__ 1
#include "zi_host.h"

extern "C" int norm_launch(const void* g, int64_t numel, int dt, int keep, uint32_t patience, void* partials, void* out)
{
    zi::NormArgs a{};
    const int64_t tiles = zi::host::NormIssuer::tiles_for((const uint16_t*)g, numel);
    a.where[0] = (uint64_t)g | (uint64_t)(tiles * zi::kNormTileElems + zi::kNormTileSlack - numel) << 48;
    a.n_tiles = (uint32_t)tiles;
    for (uint32_t& x : a.first_tile) x = 0xFFFFFFFFu;
    for (uint32_t& x : a.group_start) x = 0xFFFFFFFFu;
    a.first_tile[0] = a.group_start[0] = 0;
    a.first_tile[1] = a.n_tiles;
    a.partials = (zi::NormPartial*)partials;
    a.mark_low = 0x12345679u;
    a.mark_high = 0x9ABCDEF1u;
    a.patience = patience;
    a.out = (zi_norm_result*)out;
    a.loss_scale = 2.0f;
    const uint32_t blocks = a.n_tiles < (uint32_t)zi::kNormGroups ? a.n_tiles : (uint32_t)zi::kNormGroups;
    a.n_groups = blocks;
    return (int)zi::launch_norm_partials(a, blocks, dt, keep != 0, false, nullptr);
}
