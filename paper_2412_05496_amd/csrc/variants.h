// Table of the (mask_mod, score_mod) pairs that the forward and backward kernels are instantiated
// for.  Each pair is compiled in its own translation unit (-DFLEXATTN_VARIANT=<index>) so that the
// build can run in parallel; the dispatchers look the pair up here.
#pragma once

#include "flex_common.h"

namespace flexattn {

struct Variant {
    uint32_t mask, score;
};

#define FLEXATTN_VARIANT_ENTRY(M, S) {M, S},
constexpr Variant kVariants[] = {FLEXATTN_FOR_EACH_VARIANT(FLEXATTN_VARIANT_ENTRY)};
#undef FLEXATTN_VARIANT_ENTRY
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
#define FLEXATTN_COUNT_ONE(i) +1
static_assert(kNumVariants == 0 FLEXATTN_VARIANT_INDICES(FLEXATTN_COUNT_ONE),
              "FLEXATTN_VARIANT_INDICES (flex_common.h) and NUM_VARIANTS (build.py) must list every variant");
#undef FLEXATTN_COUNT_ONE

inline int find_variant(uint32_t mask, uint32_t score) {
    for (int i = 0; i < kNumVariants; ++i)
        if (kVariants[i].mask == mask && kVariants[i].score == score) return i;
    return -1;
}

// the variant of a call (of a valid mask).  (Forward at D = 128: cells' masks spill 16 and 28 registers more there, 469 -> 682 us)
inline int variant_of(uint32_t mask, uint32_t score, const flexattn_mod_params* p, bool backward, int D) {
    if (!mask_uses(mask, FLEXATTN_M_NEIGHBORHOOD)) return find_variant(mask, score);
    if ((backward || D == 64) && canvas_in_cells(*p)) return find_variant(mask | (p->na_layout == FLEXATTN_NA_MORTON ? kCanvasCellsZ : kCanvasCells), score);
    return find_variant(canvas_by_tags(*p, backward) ? mask | kCanvasByTags : mask, score);
}

#define FLEXATTN_CAT_(a, b) a##b
#define FLEXATTN_CAT(a, b) FLEXATTN_CAT_(a, b)

}  // namespace flexattn
