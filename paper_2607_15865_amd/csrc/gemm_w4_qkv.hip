// Prefill GEMM (gemm_w4.h), q/k/v (RoPE, cache write) epilogue.  One source per epilogue: the
// kernel's variants compile in parallel.
#include "gemm_w4.h"

int launch_gemm_w4_qkv(const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmPlan& p, const GemmShape& gs,
                      hipStream_t stream) {
    return launch_epi<EPI_QKV>(p, X, ldx, W, ep, gs, stream);
}
