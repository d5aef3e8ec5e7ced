// One launch of the reduction's kernel with a patience of the test's choice, through the library's own launcher.
#define __HIP_PLATFORM_AMD__ 1
#include "zi_host.h"

extern "C" int norm_launch(const void* g, int64_t numel, int dt, int keep, uint32_t patience, void* partials, void* out)
{
    zi::NormArgs a{};
    a.t[0] = {(const uint16_t*)g, (uint32_t)numel, 0};
    a.n_desc = 1;
    a.n_tiles = (uint32_t)zi::host::NormIssuer::tiles_for((const uint16_t*)g, numel);
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
