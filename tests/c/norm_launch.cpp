// One launch of the reduction's kernel that makes the final sum, with a patience of the test's choice, through the library's own
// launchers: `pieces` tensors of `each` elements, one behind the other, in one of the three forms of arguments.
#define __HIP_PLATFORM_AMD__ 1
#include "zi_host.h"

using zi::host::NormIssuer;

template <typename Args>
static uint32_t fill(Args& a, const uint16_t* g, int64_t each, int pieces)
{
    const int64_t tiles = NormIssuer::tiles_for(g, each);
    for (int i = 0; i < pieces; ++i) {
        a.where[i] = (uint64_t)(g + i * each) | (uint64_t)(tiles * zi::kNormTileElems + zi::kNormTileSlack - each) << 48;
        a.first_tile[i] = (uint32_t)(i * tiles);
    }
    NormIssuer::finish_list(a, pieces, (uint32_t)(pieces * tiles));
    return (uint32_t)(pieces * tiles);
}

template <typename Args>
static void common(Args& a, uint32_t tiles, uint32_t patience, void* partials, void* out, int accumulate)
{
    const uint64_t number = zi::host::next_norm_number();
    a.n_tiles = tiles;
    a.n_groups = tiles < (uint32_t)zi::kNormGroups ? tiles : (uint32_t)zi::kNormGroups;
    a.mark_low = (uint32_t)number << 1 | 1u;
    a.mark_high = (uint32_t)(number >> 31) << 1 | 1u;
    a.patience = patience;
    a.loss_scale = 2.0f;
    a.partials = (zi::NormPartial*)partials;
    a.out = (zi_norm_result*)out;
    a.accumulate = accumulate;
}

// form 0: NormArgs, 1: NormOne (one piece), 2: NormFew (keep only).  `before`: partials in front of this launch's that a launch
// before it left (form 0 only).  Whole tiles between the pieces: `each` is a multiple of 8, g 16-byte aligned.
extern "C" int norm_launch(const void* g, int64_t each, int pieces, int dt, int form, int keep, uint32_t patience, void* partials,
                           uint32_t before, void* out, int accumulate)
{
    const uint16_t* grads = (const uint16_t*)g;
    if (form == 1) {
        zi::NormOne a{};
        common(a, (uint32_t)NormIssuer::tiles_for(grads, each), patience, partials, out, accumulate);
        a.g = grads;
        a.numel = (uint32_t)each;
        return (int)zi::launch_norm_one(a, dt, keep != 0, nullptr);
    }
    if (form == 2) {
        zi::NormFew a{};
        common(a, fill(a, grads, each, pieces), patience, partials, out, accumulate);
        return (int)zi::launch_norm_few(a, dt, nullptr);
    }
    zi::NormArgs a{};
    common(a, fill(a, grads, each, pieces), patience, partials, out, accumulate);
    a.partials += before;
    a.n_before = before;
    return (int)zi::launch_norm_partials(a, a.n_groups, dt, keep != 0, false, nullptr);
}
