// The launch planners (csrc/whz_dispatch.hip) for host tests: compiled in, with
// the kernels they dispatch to as stubs that fail.
#pragma once

#include "whz_dispatch.hip"

namespace wh {
#define X(k)                                                                                                         \
    namespace nw##k {                                                                                                \
    hipError_t decode_blocks(const void*, uint64_t, uint64_t, float*, hipStream_t) { return hipErrorUnknown; }       \
    hipError_t decode_matrix(const void*, uint32_t, uint32_t, float*, hipStream_t) { return hipErrorUnknown; }       \
    hipError_t encode(const float*, uint32_t, uint32_t, void*, uint32_t*, hipStream_t) { return hipErrorUnknown; }   \
    hipError_t gemv(const GemvPlan&, AccMode, const void*, const float*, float*, double*, hipStream_t)               \
    {                                                                                                                \
        return hipErrorUnknown;                                                                                      \
    }                                                                                                                \
    hipError_t mrhs(const MrhsPlan&, const void*, const void*, uint32_t, uint32_t, float*, uint32_t, double*,        \
                    hipStream_t)                                                                                     \
    {                                                                                                                \
        return hipErrorUnknown;                                                                                      \
    }                                                                                                                \
    }
WH_FOR_EACH_NW(X)
#undef X
} // namespace wh
