// Prefill GEMM (gemm_w4.h), q/k/v (RoPE, cache write) epilogue.  One source per epilogue: the
// kernel's variants compile in parallel.
#include "gemm_w4.h"

int launch_gemm_w4_qkv(const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmPlan& p, const GemmShape& gs,
                      hipStream_t stream) {
    return launch_epi<EPI_QKV>(p, X, ldx, W, ep, gs, stream);
}

int load_gemm_w4_qkv() { return load_code((const void*)gemm_w4_kernel<EPI_QKV, 1, 2, false, WF_INT4, 4, 1>); }
