// What the few-token kernels (gemm_few.hip, attention_few.hip) share.
#pragma once
#include "sti_internal.hpp"

namespace sti {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));

// NB: room for weight blocks among the arguments (an argument list of 64 blocks costs the host 1.2 us more per launch)
template <int NB>
struct FewBlocks {
    GemmBlock b[NB];
};
}  // namespace sti
