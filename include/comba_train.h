/*
 * comba_train.h -- training entry points beside those of comba.h, for callers
 * that keep activations and their gradients in in_dtype (torch.autograd does).
 * The conventions of comba.h hold.
 */
#ifndef COMBA_TRAIN_H
#define COMBA_TRAIN_H

#include "comba.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * comba_chunk_bwd_saved with dq, dk, dv, dbeta and dbeta_tilde in in_dtype
 * instead of fp32 (bf16: the fp32 values rounded to nearest even on the way
 * out), as a model whose parameters and activations are in_dtype takes them;
 * dg, dd and dh0 stay fp32.  Alignment: dq, dk, dv 16 bytes, dbeta and
 * dbeta_tilde their element size.
 */
comba_status comba_chunk_bwd_saved_in_dtype(const comba_shape *shape, const void *q, const void *k,
                                            const void *v, const float *g, const void *beta,
                                            const void *beta_tilde, const float *d,
                                            const float *h0, const void *dO, const float *dht,
                                            void *dq, void *dk, void *dv, float *dg, void *dbeta,
                                            void *dbeta_tilde, float *dd, float *dh0, void *ws,
                                            size_t ws_bytes, void *stream);

#ifdef __cplusplus
}
#endif

#endif /* COMBA_TRAIN_H */
