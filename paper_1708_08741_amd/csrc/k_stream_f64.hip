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

hipError_t launch_parts_packed_f64(const PackTable &t, int threads, uint32_t lds, hipStream_t s) {
    return sweep::launch_parts_packed_typed<double>(t, threads, lds, s);
}

// the classification of several lattices in one dispatch, a workgroup per
// particle
__global__ void __launch_bounds__(kPartThreads) k_classify_packed(PackTable t) {
    extern __shared__ __align__(16) unsigned char part_lds[];
    const uint32_t gb = row_block();
    if (gb >= t.start[t.n]) return;
    const int e = pack_find(t, gb);
    const LatticeDev *d = t.d[e];
    const uint32_t st = t.state[e], c = st >> 1;
    ParticleArgs pa = sweep::packed_args(&d->pa);
    if (sweep::load_uniform(&d->split)) {
        pa.plist = sweep::as_global(sweep::load_uniform(&d->plist[st & 1u]));
        pa.pcount = sweep::as_global(sweep::load_uniform(&d->pcount[st & 1u]));
    }
    part::classify(pa, (int)(gb - t.start[e]), sweep::packed_args(&d->map[c]),
                   sweep::packed_args(&d->map[c == 2 ? 0 : c + 1]), part::box_rows(part_lds, pa.box_rows));
}

hipError_t launch_classify_packed(const PackTable &t, int threads, uint32_t lds, hipStream_t s) {
    const uint32_t total = t.start[t.n];
    if (t.n == 0 || total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_classify_packed, row_grid(total), dim3(threads), lds, s, t);
    return hipGetLastError();
}

int near_wall_blocks(const Grid &g, bool walls, int threads) {
    return sweep::near_wall_blocks(g.N, walls, threads);
}
uint32_t near_lds(int threads) { return sweep::near_lds_of(threads); }
uint32_t parts_blocks(int mode, int np, int wall_blocks) {
    return (uint32_t)np * (mode == kPartsSplit ? 3u : mode == kPartsClear ? 2u : 1u) + (uint32_t)wall_blocks;
}

}  // namespace lbmep
