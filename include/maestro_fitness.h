/*
 * maestro_fitness.h -- routing by fitness with caller-owned scratch.
 *
 * maestro_route_fitness (maestro.h) takes no workspace and scores every (stage, node) pair.
 * maestro_route_fitness_pruned gives the same outputs, bit for bit, from tables it builds in a
 * workspace: the nodes in ascending headroom and, per block of them, upper bounds of the fitness,
 * so that a stage scores only the nodes that can enter its result. The conventions of maestro.h
 * hold (device pointers, caller-owned arrays, asynchronous on `stream`, host-side checks first).
 */
#ifndef MAESTRO_FITNESS_H
#define MAESTRO_FITNESS_H

#include "maestro.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Workspace bytes of maestro_route_fitness_pruned, or 0 where scoring every pair is the faster
 * way by far (small batches, few nodes) or the tables are not built (more than 4,096 nodes,
 * k > 4): call maestro_route_fitness then. with_plans: nonzero when the call passes plans. */
MAESTRO_API size_t maestro_route_fitness_workspace(int64_t n, int32_t n_models, int32_t n_nodes,
                             int32_t n_src, int32_t n_classes, int32_t k, int32_t with_plans);

/* maestro_route_fitness with a workspace of at least maestro_route_fitness_workspace() bytes, 16-byte
 * aligned (MAESTRO_ERR_WORKSPACE when it is smaller; MAESTRO_ERR_UNSUPPORTED where that size is
 * 0; MAESTRO_ERR_INVALID_ARG when NULL or misaligned). Where scoring every pair is still the faster
 * way the workspace is left as it is. Other arguments, outputs and errors as
 * maestro_route_fitness; all arrays stay alive until the stream reaches the call's end. */
MAESTRO_API maestro_status maestro_route_fitness_pruned(int64_t n, const int32_t* model_id, const int32_t* src_id,
                             const int32_t* class_id, const double* kv_bytes, int32_t n_models,
                             int32_t n_nodes, int32_t n_src, int32_t n_classes,
                             const double* free_bytes, const float* queue_ms, const float* act_ms,
                             const uint64_t* resident_mask, const float* act_matrix, const float* deg_ms,
                             const maestro_deg_plan* plans, const maestro_plan_step* plan_steps,
                             const float* rtt_ms,
                             const float* class_weights, const float* bounds, double rho, int32_t k,
                             int32_t* node_idx, float* fitness, void* workspace, size_t workspace_bytes,
                             void* stream);

#ifdef __cplusplus
}
#endif

#endif /* MAESTRO_FITNESS_H */
