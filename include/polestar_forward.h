/*
 * polestar_forward.h -- calls of polestar.h run together, for forwards over
 * whole layers.  Each does what the calls it names do, under their conditions
 * and with their conventions (pointers, layouts, workspaces, errors), in fewer
 * launches and passes over memory.
 */
#ifndef POLESTAR_FORWARD_H
#define POLESTAR_FORWARD_H

#include "polestar.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * polestar_project_qkv -- polestar_refresh_kv of the rows [row_start,
 * row_start + n_rows) of every sequence (no list) and polestar_project_q of
 * the same rows as one product, for forwards whose rows are all rewritten.
 *   q : [batch][n_rows][n_heads][head_dim] dtype (output)
 *   workspace : >= polestar_project_qkv_workspace_size(...) bytes
 * Arguments and conditions otherwise as for those calls.
 */
size_t polestar_project_qkv_workspace_size(polestar_dtype dtype, int batch, int d, int n_heads,
                                           int n_kv_heads, int head_dim, int n_rows);
polestar_status polestar_project_qkv(polestar_dtype dtype, int batch, int seq, int d, int n_heads,
                                     int n_kv_heads, int head_dim, const void* h_cur, int row_start,
                                     int n_rows, const void* w_q, const void* w_k, const void* w_v,
                                     void* q, void* k_cache, void* v_cache, void* workspace,
                                     size_t workspace_bytes, hipStream_t stream);

/*
 * polestar_residual_rmsnorm -- polestar_residual_add of a whole row set, then
 * polestar_rmsnorm of the sums, in one pass with the same results:
 *   x[b][r] += y[b][r];  out[b][out_start + r] = RMSNorm(x[b][r]), r < n_rows
 *   x : [batch][n_rows][d] float, in/out;  y : [batch][n_rows][d] dtype;
 *   out : [batch][out_seq][d] dtype
 * UNSUPPORTED under polestar_rmsnorm's conditions (and y 16-byte aligned).
 */
polestar_status polestar_residual_rmsnorm(polestar_dtype dtype, int batch, int n_rows, int d, float* x,
                                          const void* y, float eps, void* out, int out_seq, int out_start,
                                          hipStream_t stream);

/*
 * polestar_linear_swiglu -- polestar_linear with W = [gate; up] ([2*ffn][n_in])
 * and polestar_swiglu of its rows: out[b][r][f] = silu(gate) * up, gate and up
 * rounded to dtype first.  gate_up [batch][n_rows][2*ffn] is scratch (the
 * product goes there where one launch does not do both); its contents are
 * undefined afterwards.
 *   workspace : >= polestar_linear_workspace_size(dtype, batch, n_rows, 2*ffn, n_in)
 * UNSUPPORTED under polestar_linear's conditions for 2*ffn outputs.
 */
polestar_status polestar_linear_swiglu(polestar_dtype dtype, int batch, int seq, int n_in, int ffn,
                                       int row_start, int n_rows, const void* x, const void* w_gate_up,
                                       void* gate_up, void* out, void* workspace, size_t workspace_bytes,
                                       hipStream_t stream);

#ifdef __cplusplus
}
#endif

#endif
