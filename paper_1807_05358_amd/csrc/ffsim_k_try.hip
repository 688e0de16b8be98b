// Trial-mutation kernels (proposals evaluated against a chain's stored timeline); compiled once
// per (FFSIM_EXT, FFSIM_GPN).
#include "ffsim_select.h"

#if !defined(FFSIM_EXT) || !defined(FFSIM_GPN)
#error "define FFSIM_EXT (0/1/2) and FFSIM_GPN (0/4)"
#endif

namespace ffsim {

template <bool WIDE, bool CACHE>
static try_kernel_t try_kernel_of(const KernelChoice& k) {
    constexpr int EXT = FFSIM_EXT;
    constexpr int GPN = FFSIM_GPN;
    return k.n_groups > FLAT_GROUPS ? k_sim_chain_try<WIDE, true, CACHE, EXT, GPN> : k_sim_chain_try<WIDE, false, CACHE, EXT, GPN>;
}

template <>
try_kernel_t try_kernels<FFSIM_EXT, FFSIM_GPN>(const KernelChoice& k) {
    // (extents that fit 16 bits without the need for 64-bit arithmetic: k_loop_chain_try)
    if (k.cache) return try_kernel_of<true, true>(k);
    return k.wide ? try_kernel_of<true, false>(k) : try_kernel_of<false, false>(k);
}

template <>
try_kernel_t loop_try_kernels<FFSIM_EXT, FFSIM_GPN>(const LoopChoice& k) {
    constexpr int EXT = FFSIM_EXT;
    constexpr int GPN = FFSIM_GPN;
    if (k.lds) {
        if (k.rowl == WAVE) return k_loop_chain_try<true, Q_OP, WAVE, EXT, GPN>;
        return k.queue == Q_OP16 ? k_loop_chain_try<true, Q_OP16, 16, EXT, GPN> : k_loop_chain_try<true, Q_OP, 16, EXT, GPN>;
    }
    return k.rowl == WAVE ? k_loop_chain_try<false, Q_SLOT, WAVE, EXT, GPN> : k_loop_chain_try<false, Q_SLOT, 16, EXT, GPN>;
}

}  // namespace ffsim
