/*
 * The weight copies of dbmp_cnn.h for several layers at once (libdiffbmp.so): what a training step
 * needs after its optimiser, in one launch instead of one per layer.
 */
#ifndef DBMP_CNN_CAST_H
#define DBMP_CNN_CAST_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* dbmp_cnn_cast_weights for each of n layers (16 to a launch). The arrays hold n entries in HOST
 * memory and may be freed when the call returns; the pointers in them are device memory. Checked
 * as a whole before anything is launched; conventions and return values as in dbmp_cnn.h. */
int dbmp_cnn_cast_layers(void *stream, int n, const float *const *w, const int *R, const int *T,
                         const int *C, uint16_t *const *wb, uint16_t *const *wt);

#ifdef __cplusplus
}
#endif

#endif /* DBMP_CNN_CAST_H */
