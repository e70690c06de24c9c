/*
 * blr_chain.h - a decoder-layer chain of BLR linears as one object: the seven linears of every layer and the glue
 * between them (blr.h), enqueued by one call.
 *
 * Wiring per layer, h the residual stream, all activations [T][hidden] or [T][mlp] in bf16:
 *     n = rmsnorm(h);  a = (W_q n + W_k n + W_v n) / sqrt(3);  h += W_o a
 *     n = rmsnorm(h);  h += W_down( silu(W_gate n) * W_up n )
 * The linears that share an input are grouped (blr_monarch_group_first_factor, blr_blast_group_forward); in a Monarch
 * chain q, k, v, gate and up leave the blocked output order, which o and down read (BLR_MONARCH_IN_BLOCKED).
 *
 * Where the kernels allow it the sum of q, k, v and the SiLU gate are computed where their last products are; with a handful of
 * tokens the norms too, inside the products behind them (two launches per linear or group, eight per layer). Every other step is a
 * call of blr.h. Results differ from those of the steps by roundings. From its second call on a chain replays its
 * launches as a HIP graph, except on a stream that is being captured; the second call captures and instantiates the graph
 * (0.6 ms of host time for 128 launches, once, 1.2 ms for 300).
 *
 * Ownership: the factors and all buffers are the caller's and must outlive the chain; the handle holds host memory and,
 * from the second call on, one HIP graph. Calls on one chain use its buffers: overlapping calls race.
 */
#ifndef BLR_CHAIN_H
#define BLR_CHAIN_H

#include "blr.h"

#ifdef __cplusplus
extern "C" {
#endif

typedef struct blr_chain blr_chain;

typedef struct {
    int blast;                       /* 0: all linears Monarch, 1: all BLAST */
    int layers;
    int64_t T;
    int hidden, mlp, b, r_square, r_mlp;
    float eps;
} blr_chain_desc;

/* The factors of one linear or group. Monarch: first (R, grouped; of o and down: re-ordered for blocked input) and second
 * (L, grouped) factor. BLAST: packed buffer and U (grouped). */
typedef struct { const void* first; const void* second; } blr_chain_factors;
typedef struct { blr_chain_factors qkv, o, gate_up, down; } blr_chain_layer;

/* Device buffers: h, h2, n, a, o, dn [T][hidden]; qkv [T][3 hidden]; gu [T][2 mlp]; m [T][mlp]; workspace: the largest of the linears (BLAST
 * beyond 4096 tokens: the smaller sizes that blr_blast_forward accepts will do). */
typedef struct {
    void *h, *h2, *n, *a, *o, *dn, *qkv, *gu, *m, *workspace;
    size_t workspace_bytes;
} blr_chain_buffers;

/* BLR_ERR_INVALID_ARG: sizes or null pointers; BLR_ERR_UNSUPPORTED: a linear or group of these shapes does not run on
 * the kernels with an intermediate in the workspace (no grouped execution, or one kernel for the whole layer). */
blr_status blr_chain_create(const blr_chain_desc* desc, const blr_chain_layer* layers, const blr_chain_buffers* buffers, blr_chain** out);
/* Runs the chain on the residual stream that h holds, in place. */
blr_status blr_chain_forward(blr_chain* chain, blr_stream stream);
/* Waits for the last pass if that was a replay of the graph. */
void blr_chain_destroy(blr_chain* chain);

#ifdef __cplusplus
}
#endif
#endif /* BLR_CHAIN_H */
