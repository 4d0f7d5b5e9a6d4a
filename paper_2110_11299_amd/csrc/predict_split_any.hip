// predict_split for projection dimensions of 80, 96 and 112 (two contraction steps).
#include "predict_split.h"

namespace dsa {

hipError_t launch_split_any(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx,
                            const AttendPtrs *attend, bool *attended, hipStream_t st)
{
    return launch_split_k<0>(sh, Qt, Kt, idx, attend, attended, st);
}

}  // namespace dsa
