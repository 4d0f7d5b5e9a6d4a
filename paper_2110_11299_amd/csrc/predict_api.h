// Host-side launchers of predict.hip and predict_split_*.hip (mask predictor, row-max contraction, MFMA yardstick): each validates nothing (the ABI layer did) and enqueues kernels.
#pragma once

#include "dsa_internal.h"

namespace dsa {

// The tensors of the attention over the mask that is predicted.
struct AttendPtrs { const void *Q, *K, *V; float *O; };
// The mask; with `attend` the same launch also computes the attention over it where that pays, and says so in *attended.
hipError_t launch_predict(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, void *ws,
                          const AttendPtrs *attend, bool *attended, hipStream_t st);
size_t predict_workspace_bytes(const dsa_shape &sh);
// Wavefronts of the workgroups of a launch_predict that have one tile of units (the attention of a tile by itself takes as many, and sums
// in the same order), 0 where they have two.
int predict_waves(const dsa_shape &sh);
hipError_t launch_rowmax(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *rowmax,
                         hipStream_t st);
hipError_t launch_mfma_i8_stream(int blocks, int iters, int32_t *sink, hipStream_t st);
// predict_split, one translation unit per projection dimension.
hipError_t launch_split_k16(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, const AttendPtrs *attend,
                            bool *attended, hipStream_t st);
hipError_t launch_split_k32(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, const AttendPtrs *attend,
                            bool *attended, hipStream_t st);
hipError_t launch_split_k48(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, const AttendPtrs *attend,
                            bool *attended, hipStream_t st);
hipError_t launch_split_k64(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, const AttendPtrs *attend,
                            bool *attended, hipStream_t st);
hipError_t launch_split_k128(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, const AttendPtrs *attend,
                            bool *attended, hipStream_t st);
hipError_t launch_split_any(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, const AttendPtrs *attend,
                            bool *attended, hipStream_t st);
// Largest L the predict kernels accept.
int predict_max_L();

}  // namespace dsa
