// predict_split for a projection dimension of 48.
#include "predict_split.h"

namespace dsa {

hipError_t launch_split_k48(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx,
                            const AttendPtrs *attend, bool *attended, hipStream_t st)
{
    return launch_split_k<48>(sh, Qt, Kt, idx, attend, attended, st);
}

}  // namespace dsa
