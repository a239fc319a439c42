// polestar_project_qkv: the K/V refresh and the Q projection of rows that are
// all rewritten, as one product of three weight matrices.  In a file of its
// own: a third matrix in the shared kernels' addressing, or its kernels in the
// code objects that a layer step launches from, slows the smallest steps (the
// tiny fp32 step 24.5 us with them there, 24.25 without).
#include "gemm_kernels.hpp"
#include "polestar_forward.h"

extern "C" size_t polestar_project_qkv_workspace_size(polestar_dtype dtype, int batch, int d, int n_heads,
                                                      int n_kv_heads, int head_dim, int n_rows) {
    using namespace ps;
    if (!dtype_ok(dtype) || batch <= 0 || d <= 0 || n_heads <= 0 || n_kv_heads <= 0 || head_dim <= 0 || n_rows <= 0)
        return 0;
    return gemm_plan(dtype == POLESTAR_BF16, static_cast<long>(batch) * n_rows,
                     (n_heads + 2 * n_kv_heads) * head_dim, d).ws_bytes;
}

extern "C" polestar_status polestar_project_qkv(polestar_dtype dtype, int batch, int seq, int d, int n_heads,
                                                int n_kv_heads, int head_dim, const void* h_cur, int row_start,
                                                int n_rows, const void* w_q, const void* w_k, const void* w_v,
                                                void* q, void* k_cache, void* v_cache, void* workspace,
                                                size_t workspace_bytes, hipStream_t stream) {
    using namespace ps;
    if (!dtype_ok(dtype) || batch <= 0 || seq <= 0 || d <= 0 || n_heads <= 0 || n_kv_heads <= 0 ||
        head_dim <= 0 || n_rows <= 0 || row_start < 0 || row_start > seq - n_rows || !h_cur || !w_q || !w_k ||
        !w_v || !q || !k_cache || !v_cache)
        return POLESTAR_ERR_INVALID_ARGUMENT;
    const bool bf16 = dtype == POLESTAR_BF16;
    if ((head_dim != 64 && head_dim != 128) || !gemm_k_ok(bf16, d) || !aligned16(h_cur) || !aligned16(w_q) ||
        !aligned16(w_k) || !aligned16(w_v) || !aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) ||
        !aligned16(workspace) || batch > 65535)
        return POLESTAR_ERR_UNSUPPORTED;
    const long m_max = static_cast<long>(batch) * n_rows;
    if (m_max > 0x7fffffffL / 4) return POLESTAR_ERR_UNSUPPORTED;
    const int kvd = n_kv_heads * head_dim;
    QkvGemmArgs g{refresh_gemm_args(batch, seq, d, kvd, h_cur, nullptr, nullptr, 0, row_start, n_rows, w_k, w_v,
                                    k_cache, v_cache, workspace),
                  static_cast<const char*>(w_q), 2 * kvd, static_cast<char*>(q)};
    g.N = 2 * kvd + n_heads * head_dim;
    const GemmPlan p = gemm_plan(bf16, m_max, g.N, d);
    if (workspace_bytes < p.ws_bytes || (p.ws_bytes > 0 && !workspace)) return POLESTAR_ERR_WORKSPACE;
    return run_plan<QkvGemmArgs>(bf16, p, g, stream, nullptr);
}
