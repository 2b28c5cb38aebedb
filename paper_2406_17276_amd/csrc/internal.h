/* Library entry points that only the Python binding and the tests use (not part of the public header). */
#pragma once

#include "opttree.h"

#ifdef __cplusplus
extern "C" {
#endif

/* ot_tree_begin that also sets the caller's frontier arrays in the same launch: token and parent slot [batch][n] to -1,
 * count [batch] to 0. */
OT_API int ot_internal_tree_begin(const ot_build_params* p, void* workspace, size_t workspace_bytes, int32_t* frontier_token,
                                  int32_t* frontier_parent_slot, int32_t* frontier_count, void* hip_stream);

/* ot_build_tree, with adapt ot_build_tree_adaptive, whose drafting workgroup waits for a row for `polls` looks at most before it
 * leaves the tree to the workgroup that scans the last row.  one_launch (host, may be null): 1 if scan and drafting are one launch. */
OT_API int ot_internal_build_tree(const ot_build_params* p, int32_t adapt, double delta, const void* logits, void* workspace,
                                  size_t workspace_bytes, const ot_tree_out* out, int32_t* steps_used, double* e_sub, int32_t polls,
                                  int32_t* one_launch, void* hip_stream);

/* How an attention call is cut up (host only): packed query rows per workgroup, key ranges per row block, whether the
 * sequences of the batch are taken longest first.  kv8: for the 8-bit cache; room: bytes of the workspace. */
OT_API int ot_internal_attn_plan(const ot_attn_params* p, int32_t kv8, size_t room, int32_t* rows, int32_t* splits, int32_t* balance);

#ifdef __cplusplus
}
#endif
