// k_stream_f64.hip -- FP64 instantiation of the fused sweep (sweep_impl.h).
// Built without floating-point contraction: the collision, forcing and
// bounce-back evaluate the same operation sequence as a plain FP64 CPU
// implementation of Sec. 3.1-3.2 of arXiv:1708.08741.
#include "near_impl.h"

namespace lbmep {

hipError_t launch_sweep_f64(int mode, int force_mode, const SweepArgs &a, int block_x,
                            const MapSetArgs *ms, hipStream_t s) {
    return sweep::launch_typed<double>(mode, force_mode, a, block_x, ms, s);
}

hipError_t launch_macro_f64(int force_mode, const SweepArgs &a, bool pull, double *rho, double *u,
                            hipStream_t s) {
    return sweep::launch_macro_typed<double>(force_mode, a, pull, rho, u, s);
}

hipError_t launch_parts_f64(const SweepArgs &a, const PartsArgs &q, hipStream_t s) {
    return sweep::launch_parts_typed<double>(a, q, s);
}

hipError_t launch_sweep_packed_f64(int force_mode, const PackTable &t, hipStream_t s) {
    return sweep::launch_sweep_packed_typed<double>(force_mode, t, s);
}

hipError_t launch_parts_packed_f64(const PackTable &t, uint32_t lds, hipStream_t s) {
    return sweep::launch_parts_packed_typed<double>(t, lds, s);
}

int near_wall_blocks(const Grid &g, bool walls) { return sweep::near_wall_blocks(g.N, walls); }
uint32_t near_lds() { return sweep::kNearLds; }
int near_blocks(int np, const Grid &g, bool walls) {
    return np + sweep::near_wall_blocks(g.N, walls);
}

}  // namespace lbmep
