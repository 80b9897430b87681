// Prefill GEMM: launch plan and dispatch (the kernel: gemm_w4.h).
#include "launch.h"

// blocks of a launch that splits k, at most
static long long max_split_blocks(int num_cus) { return num_cus * 11 / 5; }

bool gemm_w4_built(const DevLinear& W, int TM, int WN, int KG) {
    if (TM == 4) return WN == 4 && KG == 1 && !W.zeros && W.lgG != 5 && W.wf == WF_INT4;
    if (TM != 1 && TM != 2) return false;
    if (W.wf == WF_F16 && TM == 2) return WN == 4 && KG == 1;
    if (TM == 2 && WN == 2 && W.zeros && W.lgG == 5) return false;   // (would spill)
    return (WN == 4 && (KG == 1 || KG == 2)) || (WN == 2 && KG == 4);
}

GemmPlan gemm_w4_plan_of(int M, const DevLinear& W, int TM, int WN, int KG, int S) {
    GemmPlan p;
    p.TM = TM; p.WN = WN; p.KG = KG; p.S = S;
    p.nrb = (M + 32 * TM - 1) / (32 * TM);
    p.ncb = (W.N_dev + 64 * WN - 1) / (64 * WN);
    p.tiles = p.nrb * p.ncb;
    p.part_bytes = S > 1 ? (size_t)p.tiles * S * TM * 16 * WN * 64 * 8 : 0;
    return p;
}

// Launch plan: the block shape and k split with the least estimated time.
//
// The estimate (in us) counts what a CU does: its rounds of 8 waves (one block
// of 8 waves, or two of 4) times the iterations (128 k) of a wave, two more per
// round for the start of the pipeline, at the time of an iteration: 0.61 / 0.88
// / 1.33 for row tiles of 32 / 64 / 128 (a dequantised fragment serves 1, 2 or 4
// row tiles), 0.67 of it for a last round whose CUs hold one 4-wave block.  Blocks
// of 128 columns load X with two waves instead of four; k groups and k splits pay
// for the exchange of their sums.  The figures are a fit to 188 (shape, rows,
// format) points of the Llama-8B, Qwen-7B and Qwen-0.5B layers at 16 to 2011 rows,
// every plan of each timed: the plan's choice is 0.6% slower than the best one
// in the mean (at most 9%), the earlier rule (largest row tile with 0.75 tiles
// per CU, then k splits, 4-wave blocks only) was 14%.  Llama-8B at 128 rows,
// best against earlier: q/k/v 20.0 / 25.5 us, o_proj 18.5 / 19.7, gate/up
// 40.8 / 48.1, down 29.7 / 36.7 (with events around each).
//
// The 16-bit format's row tiles of 64 load X straight to LDS (4-wave blocks of
// 256 columns only); they take over where row tiles of 32 need a second round
// of blocks or read the weights from L2 many times.  Llama-8B gate/up, row tiles
// of 32 / 64: 64 rows 61 / 60 us, 100 85 / 72, 200 122 / 96, 400 185 / 149, 800
// 306 / 236; q/k/v at 200 rows 40 / 42.
//
// Row tiles of 128 (which round the scaled weight to fp16 outside q/k/v) are
// considered only from 0.75 tiles per CU on, 0.375 for k ranges of 12288 or more.
GemmPlan gemm_w4_plan(int M, const DevLinear& W, int num_cus) {
    const int its = W.K_pad / 128;
    const double wf_cost = W.wf == WF_F16 ? 1.6 : W.wf == WF_INT8 ? 1.1 : W.zeros ? 1.05 : 1.0;
    const double x_cost = W.wf == WF_INT8 ? 0.14 : 0.057;
    GemmPlan best;
    double best_cost = -1.0;
    for (int TM = 1; TM <= 4; TM *= 2)
        for (int shape = 0; shape < 3; shape++) {
            const int WN = shape == 2 ? 2 : 4, KG = shape == 0 ? 1 : shape == 1 ? 2 : 4;
            const int nrb = (M + 32 * TM - 1) / (32 * TM), ncb = (W.N_dev + 64 * WN - 1) / (64 * WN);
            if (!gemm_w4_built(W, TM, WN, KG)) continue;
            if (TM == 4) {
                const int need = W.K_pad >= 12288 ? num_cus * 3 / 2 : num_cus * 3;
                if (nrb * ncb * 4 < need) continue;
            }
            for (int S : {1, 2, 3, 4, 6, 8}) {
                const long long blocks = (long long)nrb * ncb * S;
                if (S > 1 && (its < 2 * S * KG || blocks > max_split_blocks(num_cus))) break;
                const double it = (its + S * KG - 1) / (S * KG) + 2;
                const double us = (TM == 1 ? 0.61 : TM == 2 ? (W.wf == WF_F16 ? 0.78 : 0.88) : 1.33) * wf_cost;
                const double usx = us + (WN == 2 ? x_cost * TM : 0.0);
                const long long slots = (long long)num_cus * (KG == 1 ? 2 : 1), rest = blocks % slots;
                double cost = (double)(blocks / slots) * it * usx;
                if (rest) cost += it * (KG == 1 && rest <= num_cus ? 0.67 * us : usx);
                if (S > 1) cost += 1.4 + 0.12 * S * TM * WN / KG + 0.26 * (double)blocks * TM * WN / num_cus;
                if (KG > 1) cost += 0.4 * TM * WN;
                if (best_cost < 0 || cost < best_cost) {
                    best_cost = cost;
                    best = gemm_w4_plan_of(M, W, TM, WN, KG, S);
                }
            }
        }
    return best;
}

bool gemm_w4_may_split(int M, const DevLinear& W, int num_cus) {
    const long long tiles = (long long)((M + 127) / 128) * ((W.N_dev + 255) / 256);   // the fewest (TM 4, WN 4)
    return 2 * tiles <= max_split_blocks(num_cus);
}

int launch_gemm_w4(int epi, const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmPlan& p,
                   int M, void* part, unsigned* cnt, hipStream_t stream) {
    if (p.S > 1 && (!part || !cnt)) return -1;
    // each XCD's L2 reads its share of one operand and all of the other: share
    // out the larger one (X: 2 bytes an element, W: 1/2, 1 or 2)
    const int rows = (long long)M * 4 > ((long long)W.N_dev << W.wf);
    GemmShape gs{M, p.nrb, p.ncb, p.S, W.K_pad / 64, (unsigned long long*)part, cnt, rows};
    switch (epi) {
        case EPI_QKV: return launch_gemm_w4_qkv(X, ldx, W, ep, p, gs, stream);
        case EPI_RESID: return launch_gemm_w4_resid(X, ldx, W, ep, p, gs, stream);
        case EPI_SWIGLU: return launch_gemm_w4_swiglu(X, ldx, W, ep, p, gs, stream);
        default: return -1;
    }
}
