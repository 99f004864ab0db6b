/* Entry points for the Python binding (csrc/marshal.cpp), not part of the public ABI: the public calls of the same
 * name plus `fill`.  With fill != 0 the call also clears what the public one leaves alone -- rows of sequences shorter
 * than max_seqlen: compressed keys, outputs, log-sum-exps and gradients 0, block lists -1 -- so that the binding can
 * hand it uninitialised tensors instead of filling them by launches of their own.  Every result then holds max_seqlen rows
 * per sequence (compressed keys: n_c(max_seqlen)); the public calls write rows below seqlens[b] only. */
#ifndef INFLLMV2_INTERNAL_H
#define INFLLMV2_INTERNAL_H

#include "../../include/infllmv2.h"

#ifdef __cplusplus
extern "C" {
#endif

int32_t infllmv2i_compress_keys(const infllmv2_params *prm, const infllmv2_tensor *k, const int32_t *seqlens,
                                int32_t batch, int32_t max_seqlen, int32_t n_new_tokens, const infllmv2_tensor *ck,
                                void *stream, int32_t fill);
int32_t infllmv2i_select_blocks(const infllmv2_params *prm, int32_t mode, const infllmv2_tensor *q,
                                const infllmv2_tensor *ck, const int32_t *seqlens, int32_t batch, int32_t max_seqlen,
                                int32_t *block_idx, void *workspace, size_t workspace_bytes, void *stream, int32_t fill);
int32_t infllmv2i_sparse_attn_prefill(const infllmv2_params *prm, const infllmv2_tensor *q, const infllmv2_tensor *k,
                                      const infllmv2_tensor *v, const int32_t *seqlens, int32_t batch,
                                      int32_t max_seqlen, const int32_t *block_idx, const infllmv2_tensor *out,
                                      float *lse, void *workspace, size_t workspace_bytes, void *stream, int32_t fill);
int32_t infllmv2i_sparse_attn_bwd(const infllmv2_params *prm, const infllmv2_tensor *q, const infllmv2_tensor *k,
                                  const infllmv2_tensor *v, const infllmv2_tensor *out, const infllmv2_tensor *dout,
                                  const float *lse, const int32_t *seqlens, int32_t batch, int32_t max_seqlen,
                                  const int32_t *block_idx, const infllmv2_tensor *dq, const infllmv2_tensor *dk,
                                  const infllmv2_tensor *dv, void *workspace, size_t workspace_bytes, void *stream,
                                  int32_t fill);

#ifdef __cplusplus
}
#endif
#endif /* INFLLMV2_INTERNAL_H */
