// Chain kernels (delta simulation and search steps); compiled once per (FFSIM_EXT, FFSIM_GPN).
#include "ffsim_select.h"

#if !defined(FFSIM_EXT) || !defined(FFSIM_GPN)
#error "define FFSIM_EXT (0/1/2) and FFSIM_GPN (0/4)"
#endif

namespace ffsim {

template <bool WIDE, bool CACHE>
static chain_kernel_t chain_kernel_of(const KernelChoice& k) {
    constexpr int EXT = FFSIM_EXT;
    constexpr int GPN = FFSIM_GPN;
    return k.n_groups > FLAT_GROUPS ? k_sim_chain_steps<WIDE, true, CACHE, EXT, GPN> : k_sim_chain_steps<WIDE, false, CACHE, EXT, GPN>;
}

template <>
chain_kernel_t chain_kernels<FFSIM_EXT, FFSIM_GPN>(const KernelChoice& k) {
    // (extents that fit 16 bits without the need for 64-bit arithmetic: k_loop_chain_steps)
    if (k.cache) return chain_kernel_of<true, true>(k);
    return k.wide ? chain_kernel_of<true, false>(k) : chain_kernel_of<false, false>(k);
}

template <>
chain_kernel_t loop_chain_kernels<FFSIM_EXT, FFSIM_GPN>(const LoopChoice& k) {
    constexpr int EXT = FFSIM_EXT;
    constexpr int GPN = FFSIM_GPN;
    if (k.lds) {
        if (k.rowl == WAVE) return k_loop_chain_steps<true, Q_OP, WAVE, EXT, GPN>;
        return k.queue == Q_OP16 ? k_loop_chain_steps<true, Q_OP16, 16, EXT, GPN> : k_loop_chain_steps<true, Q_OP, 16, EXT, GPN>;
    }
    return k.rowl == WAVE ? k_loop_chain_steps<false, Q_SLOT, WAVE, EXT, GPN> : k_loop_chain_steps<false, Q_SLOT, 16, EXT, GPN>;
}

}  // namespace ffsim
