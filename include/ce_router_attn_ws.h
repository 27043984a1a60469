/*
 * Routed attention with a caller-owned workspace, beside ce_router.h (which
 * holds every other entry point, the types and the status codes).
 */
#ifndef CE_ROUTER_ATTN_WS_H
#define CE_ROUTER_ATTN_WS_H

#include "ce_router.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * ce_routed_attention with a workspace, which decode steps over long caches
 * use: with few queries per sequence the keys of a sequence are then shared by
 * several workgroups, whose results a second launch combines in a fixed order
 * (deterministic; section 3.4, compressed key-value cache). Same arguments,
 * results and errors otherwise.
 *   ws  device workspace of ce_attention_workspace_size(attn) bytes, 256-byte
 *       aligned, contents on entry do not matter; NULL is ce_routed_attention.
 *       CE_ERR_WORKSPACE if it is short or misaligned.
 * ce_attention_workspace_size depends on the sizes in attn only (no device
 * pointer is read), is at most 17 MB, and is 0 when no workspace is used or the
 * call would refuse attn.
 */
size_t ce_attention_workspace_size(const ce_attn* attn);
int ce_routed_attention_ws(const ce_attn* attn, const void* q, const void* k, const void* v, void* o, void* ws,
                           size_t ws_bytes, void* stream);

#ifdef __cplusplus
}
#endif

#endif /* CE_ROUTER_ATTN_WS_H */
