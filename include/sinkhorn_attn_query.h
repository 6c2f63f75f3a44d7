/*
 * sinkhorn_attn_query.h -- how the library would run a call: host-only, no GPU call, nothing of the operator.  For
 * benchmarks, which price the kernels a call launches, and for tests.
 */
#ifndef SINKHORN_ATTN_QUERY_H
#define SINKHORN_ATTN_QUERY_H

#include <stddef.h>

#ifdef __cplusplus
extern "C" {
#endif

/*
 * The Sinkhorn steps after the first one of a forward (one_call 0), or of the forward half of sinkhorn_attn_step
 * (one_call 1), with a workspace of workspace_bytes; lengths: 1 if the call gives any.
 */
typedef struct {
    int whole_steps;       /* 1: a step is one launch; 0: two half-steps                                           */
    int half_steps_fuse;   /* 1: sinkhorn_attn_set_fused_half_steps applies (outside capture, without a continuation */
                           /* schedule, on a device that holds the launch); 0 where steps are whole                 */
                           /* the rest is about whole steps, 0 otherwise:                                          */
    int block_rows;        /* rows a workgroup owns at a time                                                    */
    int segment_blocks;    /* blocks a workgroup walks one after the other, at most                              */
    int segments;          /* workgroups per problem                                                             */
    int sums_apart;        /* 1: no problem's column sums lie where another problem's backward writes (if not, a  */
                           /* one-call step joins its two streams between the directions)                        */
    size_t sums_offset[2]; /* the two buffers of column sums: bytes from the workspace's start ...                */
    size_t sums_stride;    /* ... and between problems                                                           */
    size_t sums_bytes;     /* used of that, per problem                                                          */
} ska_step_plan;

/* Returns SKA_OK, or the error that the call itself would return for these sizes. */
int ska_query_step_plan(int B, int H, int L, int d, int W, int T, int R, int dustbin, int lengths, int dtype,
                        size_t workspace_bytes, int one_call, ska_step_plan *plan);

/*
 * Chains: launches whose workgroups wait for each other.  Short calls run the steps after the first one in one launch, whose
 * workgroups hand their sums to each other; sinkhorn_attn_set_fused_half_steps runs half-steps so.  They are numbered from 1
 * on, per device; the device writes `started` and `given_up` (ask after a synchronisation).
 */
typedef struct {
    unsigned launched;  /* number of the latest chain (0: there was none)                                             */
    unsigned started;   /* of the latest one whose workgroups have all started                                     */
    unsigned given_up;  /* of the latest one in which a wait has run out, 0: none (steps: they were solved again;    */
                        /* half-steps: what depends on the wait is NaN)                                        */
} ska_chains;

/* Returns SKA_OK, or SKA_EINVAL without a place for the answer or for a device number out of range. */
int ska_query_chains(int device, ska_chains *chains);

#ifdef __cplusplus
}
#endif
#endif /* SINKHORN_ATTN_QUERY_H */
