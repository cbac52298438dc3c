// k_stream_lp.hip -- FP32 and FP16 deviation-storage instantiations of the
// fused sweep (sweep_impl.h), FP32 arithmetic, and the precision dispatch of
// the sweep launch.
#include "near_impl.h"

namespace lbmep {

hipError_t launch_sweep_f64(int mode, int force_mode, const SweepArgs &a, int block_x,
                            const MapSetArgs *ms, hipStream_t s);

hipError_t launch_sweep(int precision, int mode, int force_mode, const SweepArgs &a, int block_x,
                        const MapSetArgs *ms, hipStream_t s) {
    if (precision == LBMEP_FP64) return launch_sweep_f64(mode, force_mode, a, block_x, ms, s);
    if (precision == LBMEP_FP32DEV)
        return sweep::launch_typed<float>(mode, force_mode, a, block_x, ms, s);
    return sweep::launch_typed<__half>(mode, force_mode, a, block_x, ms, s);
}

hipError_t launch_macro_f64(int force_mode, const SweepArgs &a, bool pull, double *rho, double *u,
                            hipStream_t s);

hipError_t launch_macro(int precision, int force_mode, const SweepArgs &a, bool pull, double *rho,
                        double *u, hipStream_t s) {
    if (precision == LBMEP_FP64) return launch_macro_f64(force_mode, a, pull, rho, u, s);
    if (precision == LBMEP_FP32DEV)
        return sweep::launch_macro_typed<float>(force_mode, a, pull, rho, u, s);
    return sweep::launch_macro_typed<__half>(force_mode, a, pull, rho, u, s);
}

hipError_t launch_parts_f64(const SweepArgs &a, const PartsArgs &q, hipStream_t s);

hipError_t launch_parts(int precision, const SweepArgs &a, const PartsArgs &q, hipStream_t s) {
    if (precision == LBMEP_FP64) return launch_parts_f64(a, q, s);
    if (precision == LBMEP_FP32DEV) return sweep::launch_parts_typed<float>(a, q, s);
    return sweep::launch_parts_typed<__half>(a, q, s);
}

hipError_t launch_sweep_packed_f64(int force_mode, const PackTable &t, hipStream_t s);
hipError_t launch_parts_packed_f64(const PackTable &t, int threads, uint32_t lds, hipStream_t s);

hipError_t launch_sweep_packed(int precision, int force_mode, const PackTable &t, hipStream_t s) {
    if (precision == LBMEP_FP64) return launch_sweep_packed_f64(force_mode, t, s);
    if (precision == LBMEP_FP32DEV) return sweep::launch_sweep_packed_typed<float>(force_mode, t, s);
    return sweep::launch_sweep_packed_typed<__half>(force_mode, t, s);
}

hipError_t launch_parts_packed(int precision, const PackTable &t, int threads, uint32_t lds,
                               hipStream_t s) {
    if (precision == LBMEP_FP64) return launch_parts_packed_f64(t, threads, lds, s);
    if (precision == LBMEP_FP32DEV)
        return sweep::launch_parts_packed_typed<float>(t, threads, lds, s);
    return sweep::launch_parts_packed_typed<__half>(t, threads, lds, s);
}

}  // namespace lbmep
