// Entry to the matrix-core step's launchers, one per (BATCH, RULE, AL), each
// defined in its own build of matrix_inst.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "params.hpp"

namespace nbb {

template <bool BATCH, int RULE, int AL>
hipError_t launch_matrix_inst(const MatParams &E, uint32_t nr, uint32_t nh, uint32_t gpw, const uint8_t *in,
                              uint8_t *out, uint32_t rule, const uint32_t *rec, int cu_count, hipStream_t st);
template <bool BATCH, int RULE, int AL>
hipError_t launch_hold_inst(const HoldParams &E, uint32_t nr, uint32_t nh, uint32_t gpw, uint8_t *in,
                            uint8_t *out, uint32_t rule, uint32_t gens, const uint32_t *rec, const uint32_t *steps_of,
                            uint32_t launch, uint32_t mode, hipStream_t st);

#define NBB_MAT_INST_DECL(B, R, AL)                                                                             \
    extern template hipError_t launch_matrix_inst<B, R, AL>(const MatParams &, uint32_t, uint32_t, uint32_t,    \
                                                            const uint8_t *, uint8_t *, uint32_t,               \
                                                            const uint32_t *, int, hipStream_t);            \
    extern template hipError_t launch_hold_inst<B, R, AL>(const HoldParams &, uint32_t, uint32_t, uint32_t,     \
                                                          uint8_t *, uint8_t *, uint32_t, uint32_t,             \
                                                          const uint32_t *, const uint32_t *, uint32_t,         \
                                                          uint32_t, hipStream_t);
#define NBB_MAT_INST_DECLS(B, R) \
    NBB_MAT_INST_DECL(B, R, 1)   \
    NBB_MAT_INST_DECL(B, R, 4)   \
    NBB_MAT_INST_DECL(B, R, 16)
NBB_MAT_INST_DECLS(false, 0)
NBB_MAT_INST_DECLS(false, 1)
NBB_MAT_INST_DECLS(true, 0)
NBB_MAT_INST_DECLS(true, 1)
#define NBB_HOLD_PACKED_DECL(R)                                                                                \
    extern template hipError_t launch_hold_inst<false, R, 0>(const HoldParams &, uint32_t, uint32_t, uint32_t,  \
                                                             uint8_t *, uint8_t *, uint32_t, uint32_t,          \
                                                             const uint32_t *, const uint32_t *, uint32_t,      \
                                                             uint32_t, hipStream_t);
NBB_HOLD_PACKED_DECL(0)
NBB_HOLD_PACKED_DECL(1)
#undef NBB_HOLD_PACKED_DECL
#undef NBB_MAT_INST_DECLS
#undef NBB_MAT_INST_DECL

}  // namespace nbb
