// pa_quad_any.hip -- the quad sweep kernels of the lattice sides without a
// table entry, a quarter of them (L / 2 = PA_PART mod 4) per compilation.
#include "pa_quad.h"

namespace pa {

namespace {

// Sides with tabulated lane choices have kernels of their own (pa_kernels.hip).
constexpr bool has_lane_choices(uint32_t L) {
    for (uint32_t s : {4u, 8u, 12u, 16u, 20u, 24u, 32u, 48u, 64u, 96u, 128u, 192u, 256u})
        if (s == L) return true;
    return false;
}

template <uint32_t L0>
void *instance(uint32_t L, bool batch) {
    if constexpr (L0 > 254) {
        return nullptr;
    } else {
        if constexpr (!has_lane_choices(L0))
            if (L == L0) return batch ? (void *)k_sweep_any_batch<L0> : (void *)k_sweep_any<L0>;
        return instance<L0 + 8>(L, batch);
    }
}

}  // namespace

#if PA_PART == 0
void *quad_any_part0(uint32_t L, bool batch) { return instance<8>(L, batch); }
#elif PA_PART == 1
void *quad_any_part1(uint32_t L, bool batch) { return instance<10>(L, batch); }
#elif PA_PART == 2
void *quad_any_part2(uint32_t L, bool batch) { return instance<12>(L, batch); }
#else
void *quad_any_part3(uint32_t L, bool batch) { return instance<14>(L, batch); }
#endif

}  // namespace pa
