// Full simulations for searches that look ahead; compiled once per (FFSIM_EXT, FFSIM_GPN).
#include "ffsim_select.h"

#if !defined(FFSIM_EXT) || !defined(FFSIM_GPN)
#error "define FFSIM_EXT (0/1/2) and FFSIM_GPN (0/4)"
#endif

namespace ffsim {

template <>
nodes_kernel_t loop_nodes_kernels<FFSIM_EXT, FFSIM_GPN>(const LoopChoice& k) {
    constexpr int EXT = FFSIM_EXT;
    constexpr int GPN = FFSIM_GPN;
    if (k.lds) {
        if (k.rowl == WAVE) return k_loop_nodes<true, Q_OP, WAVE, EXT, GPN>;
        return k.queue == Q_OP16 ? k_loop_nodes<true, Q_OP16, 16, EXT, GPN> : k_loop_nodes<true, Q_OP, 16, EXT, GPN>;
    }
    return k.rowl == WAVE ? k_loop_nodes<false, Q_SLOT, WAVE, EXT, GPN> : k_loop_nodes<false, Q_SLOT, 16, EXT, GPN>;
}

}  // namespace ffsim
