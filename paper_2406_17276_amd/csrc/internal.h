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

/* How an attention call is cut up (host only): packed query rows per workgroup, key ranges per row block, whether the
 * sequences of the batch are taken longest first.  kv8: for the 8-bit cache; room: bytes of the workspace. */
OT_API int ot_internal_attn_plan(const ot_attn_params* p, int32_t kv8, size_t room, int32_t* rows, int32_t* splits, int32_t* balance);

#ifdef __cplusplus
}
#endif
