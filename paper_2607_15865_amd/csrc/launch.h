// Kernel launchers (internal).
#pragma once
#include "common.h"

// Prefill GEMM launch plan: row tile (32 * TM rows), block shape (WN waves
// side by side, 64 columns each; KG groups of them that share out the block's
// k range), k splits S, grid.
struct GemmPlan {
    int TM = 4, WN = 4, KG = 1, S = 1, nrb = 0, ncb = 0, tiles = 0;
    size_t part_bytes = 0;        // fp32 partial sums (S > 1)
};
GemmPlan gemm_w4_plan(int M, const DevLinear& W, int num_cus);
// the kernel variants that exist, and the plan of a given shape
bool gemm_w4_built(const DevLinear& W, int TM, int WN, int KG);
GemmPlan gemm_w4_plan_of(int M, const DevLinear& W, int TM, int WN, int KG, int S);
// false: no plan of M rows or more splits k
bool gemm_w4_may_split(int M, const DevLinear& W, int num_cus);
// part: plan.part_bytes of workspace; cnt: plan.tiles arrival counters, zeroed
// by an earlier launch on the stream (launch_rmsnorm) and used by this launch
// alone.  Both are unused when plan.S == 1.
int launch_gemm_w4(int epi, const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmPlan& plan,
                   int M, void* part, unsigned* cnt, hipStream_t stream);

// (the kernel's launchers, one source per epilogue)
struct GemmShape {
    int M, nrb, ncb, S, KB;
    unsigned long long* part;    // [nrb * ncb][S][TM * 16][WN][64] partial pairs (S > 1)
    unsigned* cnt;               // [nrb * ncb] arrival counters, zeroed by an earlier launch (S > 1)
    int rows;                    // blocks in row order (else in column order)
};

int launch_gemm_w4_qkv(const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmPlan& plan,
                       const GemmShape& gs, hipStream_t stream);
int launch_gemm_w4_resid(const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmPlan& plan,
                         const GemmShape& gs, hipStream_t stream);
int launch_gemm_w4_swiglu(const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmPlan& plan,
                          const GemmShape& gs, hipStream_t stream);

struct GemvArgs {
    DevLinear W;
    const float* x_f32;      // NORM prologue input fp32 [B][K] (K = hidden)
    const uint16_t* gamma;   // bf16 bits [K]
    float eps;
    const f16* x_f16;        // activation input [B][ldx] (non-NORM)
    int ldx;
    int B;
    int ksplit;              // blocks along K
    int ct;                  // residual: column tiles per block (1 or 2)
    int num_cus;             // of the device: the block shape
    int off_red;             // set by the launcher
    EpiArgs ep;
    float* clear;            // fp32 words that the launch sets to zero (the output that a later
    int nclear;              // launch adds into), nclear of them
    unsigned* zero;          // words that the launch sets to zero (arrival counters of a later
    int nzero;               // launch), nzero of them
};
// Weights that a GEMV block reads: those of ct column tiles from `tile` on, one
// contiguous run of `bytes` from byte `first` of the matrix.  A block's buffer
// covers just its run, so that its 32-bit offsets do not depend on the size of
// the matrix (16-bit gate/up of hidden 16384, FFN 65536: exactly 4 GiB).
struct GemvRun {
    uint64_t first;
    uint32_t bytes;
};
constexpr uint32_t kGemvPastEnd = 0xFFFF0000u;   // an offset past every block's run
__host__ __device__ inline GemvRun gemv_run_bytes(int tile, int ct, int K_pad, int wf) {
    const uint32_t strip = (uint32_t)(K_pad / 64) << (10 + wf);     // one column tile
    return GemvRun{(uint64_t)(uint32_t)tile * strip, (uint32_t)ct * strip};
}
// the fused RMSNorm of B rows of K fits the GEMV block's registers
bool gemv_norm_fits(int B, int K);
// sets ct and ksplit of a residual GEMV (from W, B, num_cus)
void gemv_resid_plan(GemvArgs& a, bool ordered);
int launch_gemv_w4(int epi, bool norm, const GemvArgs& a, hipStream_t stream);

// zero, nzero: words that the launch also sets to zero (arrival counters of
// later launches), or null
int launch_rmsnorm(const float* x, const uint16_t* gamma, float eps, int M, int H, f16* out, int* err,
                   hipStream_t stream, unsigned* zero = nullptr, int nzero = 0);

struct AttnPrefillArgs {
    const uint16_t* q;       // bf16 [T][nq][d]
    const uint16_t* k_cache; // bf16 [nkv][max_seq][d] of the sequence
    const uint16_t* v_cache;
    long long cache_stride_h;
    f16* out;                // [T][nq*d]
    int T, L, nq, nkv, d;
    float scale_log2;        // log2(e) / sqrt(d)
    float* part;             // chunk partial states (plan.part_bytes)
    int chunk_keys, ngrp, items;   // set by the launcher from the plan
    int* err;                // the layer's error flag (W4_FLAG_F16_RANGE)
};
// Prefill attention launch plan: key chunk length, work items per block
// row, block size, workspace.
struct AttnPrefillPlan {
    int chunk_keys = 0, items = 0, ngrp = 1, threads = 64;
    bool merge = false;      // some query tile has more than one chunk
    size_t part_bytes = 0;
    size_t part_bound = 0;   // part_bytes of any history up to L (non-decreasing in L)
    size_t lds_bytes = 0;
};
AttnPrefillPlan attn_prefill_plan(int T, int L, int nq, int nkv, int d, int num_cus);
int launch_attn_prefill(const AttnPrefillArgs& a, const AttnPrefillPlan& p, hipStream_t stream);

struct AttnDecodeArgs {
    const uint16_t* q;       // bf16 [B][nq][d]
    const uint16_t* k_cache; // bf16 [B][nkv][max_seq][d]
    const uint16_t* v_cache;
    long long stride_b, stride_h;
    const int32_t* ctx_lens; // [B] device, or null: row b's context is ctx_base + b
    int ctx_base;
    const float* mask;       // [B][max_seq] or null
    int max_seq;
    float* part;             // share states, B * nq * nsplit * (d + 2) floats (nsplit > 1)
    unsigned* cnt;           // [B][nkv] arrival counters, zeroed by an earlier launch (nsplit > 1)
    f16* out;                // [B][nq*d]
    int B, nq, nkv, d, nsplit;   // nsplit: shares of a (row, kv head)'s keys
    float scale_log2;
    int* err;                // the layer's error flag (W4_FLAG_F16_RANGE)
};
int attn_decode_splits(int B, int nkv, int max_ctx, int num_cus);
int launch_attn_decode(const AttnDecodeArgs& a, hipStream_t stream);

int launch_kv_append(uint16_t* k_cache, uint16_t* v_cache, const uint16_t* k_new, const uint16_t* v_new,
                     int B, int T, int nkv, int d, long long stride_b, long long stride_h,
                     const int32_t* slot_start_host, hipStream_t stream);

int launch_debug_dequant(const DevLinear& W, const int32_t* col_map, int K, int N, float* out,
                         hipStream_t stream);

// load_code of each source
int load_gemm_w4_qkv();
int load_gemm_w4_resid();
int load_gemm_w4_swiglu();
int load_gemv_w4();
int load_attention();
int load_misc();
int load_decode_fused();
int load_lm();
