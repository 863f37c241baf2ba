/* Entry point of libnoble.so for the torch binding beside the public ones of
 * noble.h. */
#ifndef NOBLE_BINDING_H
#define NOBLE_BINDING_H

#include "noble.h"

#ifdef __cplusplus
extern "C" {
#endif

/* noble_linear_bwd with the gradients of the storage parameters (dW, dW_down,
 * dM, dW_up) in the storage dtype: the float32 sums of noble_linear_bwd rounded
 * once.  With a one-application activation a given dM, in the storage dtype too,
 * is set to zero.  T = 0 is refused on the bf16 path (NOBLE_ERR_BAD_SHAPE). */
noble_status noble_linear_bwd_storage(const noble_linear_desc* desc, const void* dy, const void* x, const void* W,
                                      const void* W_down, const float* omega1, const float* phi1, const void* M,
                                      const float* omega2, const float* phi2, const void* W_up, const void* reserve,
                                      void* dx, void* dW, float* db, void* dW_down, void* dM, void* dW_up,
                                      float* domega1, float* dphi1, float* domega2, float* dphi2, void* scratch,
                                      size_t scratch_bytes, void* stream);

#ifdef __cplusplus
}
#endif

#endif
