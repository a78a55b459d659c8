// One (BATCH, RULE, AL) combination of the matrix-core step's launchers, chosen
// by NBB_INST_BATCH (0/1), NBB_INST_RULE (0: B3/S23, 1: any rule) and
// NBB_INST_AL (1, 4 or 16; 0: the bit-packed held step alone); the build
// compiles this file once per combination.
#include "matrix.hpp"
#include "matrix_launch.hpp"

#if !defined(NBB_INST_BATCH) || !defined(NBB_INST_RULE) || !defined(NBB_INST_AL)
#error "matrix_inst.hip needs NBB_INST_BATCH, NBB_INST_RULE and NBB_INST_AL"
#endif

namespace nbb {

#if NBB_INST_AL != 0
template <bool BATCH, int RULE, int AL>
hipError_t launch_matrix_inst(const MatParams &E, uint32_t nr, uint32_t nh, uint32_t gpw, const uint8_t *in,
                              uint8_t *out, uint32_t rule, const uint32_t *rec, int cu_count, hipStream_t st) {
    return launch_matrix_shape<AL, BATCH, RULE>(E, nr, nh, gpw, in, out, rule, rec, cu_count, st);
}

template hipError_t launch_matrix_inst<bool(NBB_INST_BATCH), NBB_INST_RULE, NBB_INST_AL>(
    const MatParams &, uint32_t, uint32_t, uint32_t, const uint8_t *, uint8_t *, uint32_t, const uint32_t *, int,
    hipStream_t);
#endif

template <bool BATCH, int RULE, int AL>
hipError_t launch_hold_inst(const HoldParams &E, uint32_t nr, uint32_t nh, uint32_t gpw, uint8_t *in,
                            uint8_t *out, uint32_t rule, uint32_t gens, const uint32_t *rec, const uint32_t *steps_of,
                            uint32_t launch, uint32_t mode, hipStream_t st) {
    return launch_hold_shape<AL, BATCH, RULE>(E, nr, nh, gpw, in, out, rule, gens, rec, steps_of, launch, mode, st);
}

template hipError_t launch_hold_inst<bool(NBB_INST_BATCH), NBB_INST_RULE, NBB_INST_AL>(
    const HoldParams &, uint32_t, uint32_t, uint32_t, uint8_t *, uint8_t *, uint32_t, uint32_t, const uint32_t *,
    const uint32_t *, uint32_t, uint32_t, hipStream_t);

}  // namespace nbb
