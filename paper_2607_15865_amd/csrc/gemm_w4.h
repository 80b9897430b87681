// W4A16 GEMM for the prefill stages: Y[M][N] = X[M][K] * W[K][N] on the
// 32x32x16 fp16 MFMA with fp32 accumulation.
//
// X is an activation already rounded to bf16 and held as fp16 (exact), so the
// MFMA sees exactly the W4BF16 operand values.  W is used exactly: the B
// fragment of every k16 step is (code - zero) as fp16 integers (dequant8) and
// the group scale is applied in fp32.  The scale is carried as a running
// ratio: the accumulator u holds sum_g s_g T_g / s_cur, and at the start of
// group g it is multiplied by s_{g-1} / s_g, so one VALU multiply per output
// per group and no second accumulator set are needed; the epilogue multiplies
// by the scale of the last group of the k range.  (Rounding the scaled weight
// to fp16 instead would save those multiplies, but its 2^-12 relative error
// flips the bf16 rounding of q/k/v and of the SwiGLU output often enough to
// break the parity bound on full-size layers.)
//
// Block: WN waves side by side along N (64 columns each) times KG k groups
// (64 WN KG threads).  Block tile BM x 64 WN with BM = 32 * TM; wave tile BM x
// 64 (TM x 2 MFMA tiles), so a wave's two 32-column weight tiles are a RoPE
// pair or a gate/up pair and every dequantised weight fragment feeds TM
// MFMAs.  The k groups share out the block's k range, each with X tiles of
// its own, and exchange their sums through LDS at the end: 8 waves (two per
// SIMD, which hide each other's LDS and memory latency) work on an output
// tile where few tiles would leave the SIMDs with one wave or none, without
// the partial sums in memory that a k split over blocks costs.  Shapes
// (WN, KG): (4, 1), (4, 2), (2, 4).
//
// Pipeline, per iteration of BK = 128 k (two 64-k weight tiles per column).
// The X tile (BM x 128 fp16) lies in LDS, two buffers in turn; its rows are 256
// bytes without padding, and the 16-byte chunk c of row r is stored at chunk
// c ^ (r & 15), so the A-fragment reads of 16 consecutive rows hit 16 different
// bank groups.  Each wave holds its weight tiles (4 per iteration; 1 KB with 4
// bits, one 16-byte load per lane) in registers.  Two forms:
//   * row tiles of 32 and 64 (XREG): X and weights are requested P = 2 to 4
//     iterations ahead into P register stages; at the end of an iteration the
//     next one's X goes from its stage to LDS, and the barrier waits for
//     LDS writes only, so the deeper loads stay in flight;
//   * row tiles of 128, and of 64 with 16-bit weights: X goes straight from
//     memory to LDS (direct-to-LDS loads, 1 KB per 4 rows, no registers), one
//     iteration ahead, with the weights; the barrier's workgroup release waits
//     for the block's outstanding loads.  The scale ratio that the accumulators
//     take at the end of an iteration (the next one's first group) is
//     requested two iterations ahead.
// In both, the A fragments (LDS) and B fragments of step t + 1 are prepared
// while the MFMAs of step t run, and no instruction of an iteration waits for
// that iteration's loads.  Every load is issued unconditionally with clamped
// addresses (X rows past M read row M - 1; their outputs are dropped).  K_pad
// is a multiple of 128, so every k range holds whole iterations.
//
// Split K: with S > 1 the k tiles are cut into S ranges, one block each.
// Every block stores its fp32 partial tile, and the last block of a tile to
// arrive (a per-tile counter in the caller's workspace, zeroed by the RMSNorm
// launch that starts the call) adds the S partials in range order and runs
// the epilogue, so the result does not depend on the arrival order.
//
// Block order: consecutive block ids go round robin over the 8 XCDs, and each
// XCD takes one run of the blocks.  In column order the blocks of one column
// block (its row blocks and k ranges) share an XCD, so each weight column block
// is read from HBM into one L2 and X into all eight; where X is the larger
// operand (long prompts) the runs are in row order instead.
#pragma once
#include "common.h"
#include "launch.h"

namespace {

constexpr int NXCD = 8;

// Instruction order of one k16 step for the scheduler: every MFMA is
// followed by an LDS read of the next step's A fragments (the first TM of
// them) and a few VALU operations (dequantisation of the next step).
template <int TM, int NVALU>
__device__ __forceinline__ void sched_step() {
#pragma unroll
    for (int j = 0; j < 2 * TM; j++) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
        if (j < TM) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS read
        __builtin_amdgcn_sched_group_barrier(0x002, NVALU, 0);   // VALU
    }
}

// LDS of a block: two X tiles per k group, later the sums that the k groups
// exchange
template <int TM, int WN, int KG>
constexpr size_t lds_bytes() {
    const size_t x = (size_t)KG * 2 * 32 * TM * 256, ex = (size_t)(KG - 1) * WN * 16 * TM * 512;
    return x > ex ? x : ex;
}

// k range of part sp of S in 64-k tiles; inner split points are even so that
// iterations hold whole tile pairs (with fewer pairs than parts some are empty)
__host__ __device__ inline void split_range(int sp, int S, int KB, int& lo, int& hi) {
    const int pairs = KB / 2;
    lo = (int)((long long)sp * pairs / S) * 2;
    hi = sp == S - 1 ? KB : (int)((long long)(sp + 1) * pairs / S) * 2;
}

// GT: group size class, 0 = groups of 32 (two per 64-k tile), 1 = groups of
// 64, 2 = groups of 128 or more (starting only at the first tile of an
// iteration); ZP: the linear has zero points; WF: weight format
// (WeightFormat).  The 8- and 16-bit formats differ only in the tile bytes
// (2 or 4 quads of 16 bytes per lane) and the fragment unpack (dequant8_u8,
// f16_frag); with one scale and zero point per column they need no ratios
// (leaving out the multiplications by 1: INT8 Llama-8B, 800 rows, 496 -> 448 us
// a layer, bf16 at 64 rows 144.5 -> 141.8).
template <int EPI, int TM, int GT, bool ZP, int WF, int WN, int KG>
__global__ void __launch_bounds__(64 * WN * KG) __attribute__((amdgpu_waves_per_eu(2)))
gemm_w4_kernel(const f16* __restrict__ X, int ldx, DevLinear W, EpiArgs ep, GemmShape gs) {
    constexpr int BM = 32 * TM;
    constexpr int XL = BM / (4 * WN);                   // X loads (1 KB) per wave and iteration
    constexpr int NH = GT == 0 ? 2 : 1;                 // group parameters per tile
    constexpr bool XREG = TM < 4 && !(TM == 2 && WF == WF_F16);
    static_assert(XREG || (WN == 4 && KG == 1), "X straight to LDS: four waves side by side");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ unsigned last_flag;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wid % WN, kg = wid / WN;           // column strip, k group
    const int h = lane >> 5, c = lane & 31;
    const int M = gs.M;
    unsigned char* const As0 = smem + kg * 2 * BM * 256;
    unsigned char* const As1 = As0 + BM * 256;

    // block -> (column block, row block, k range), every XCD one run of the
    // blocks: in column order, so that a column block's weights enter one L2
    // and X all of them, or (rows) in row order, the other way round
    int cb, rb, sp;
    {
        const int xcd = blockIdx.x % NXCD, n = gridDim.x, q = n / NXCD, rem = n % NXCD;
        const int pos = xcd * q + (xcd < rem ? xcd : rem) + blockIdx.x / NXCD;
        if (gs.rows) {
            cb = pos % gs.ncb;
            const int j = pos / gs.ncb;
            sp = j % gs.S;
            rb = j / gs.S;
        } else {
            rb = pos % gs.nrb;
            const int j = pos / gs.nrb;
            sp = j % gs.S;
            cb = j / gs.S;
        }
    }
    const int m0 = rb * BM;
    const int nt0 = (cb * WN + wave) * 2;               // first of this wave's two column tiles
    const bool wave_on = nt0 * 32 < W.N_dev;            // columns past N_dev: the wave computes on
                                                        // tile 0 and stores nothing
    const int KB = gs.KB;
    int kb_lo, kb_hi;
    split_range(sp * KG + kg, gs.S * KG, KB, kb_lo, kb_hi);
    // iterations of the block's longest k group (all its waves meet in every barrier)
    const int nit = XREG ? (KB / 2 + gs.S * KG - 1) / (gs.S * KG) : (kb_hi - kb_lo) / 2;
    const int Gm1 = (1 << W.lgG) - 1;
    const int col0 = (wave_on ? nt0 : 0) * 32 + c, col1 = col0 + 32;
    const DqConst dq = dq_const();

    // ---- X tile of the iteration that starts at 64-k tile kb, to LDS: load i
    // of wave w fills rows 4 (WN i + w) .. + 3; lane L writes chunk L & 15 of
    // row 4 (WN i + w) + L / 16, which holds logical chunk (L & 15) ^ (row & 15).
    const uint32_t xrow_bytes = (uint32_t)ldx * 2u;
    const char* const Xb = reinterpret_cast<const char*>(X);
    uint32_t xoff[XL];                                  // per load: row offset + chunk (bytes)
#pragma unroll
    for (int i = 0; i < XL; i++) {
        const int r = 4 * (WN * i + wave) + (lane >> 4);
        const int m = m0 + r < M ? m0 + r : M - 1;
        xoff[i] = (uint32_t)m * xrow_bytes + (uint32_t)((lane & 15) ^ (r & 15)) * 16u;
    }
    // Pipeline depth P: the loads of iteration it + P are requested in
    // iteration it.  Row tiles of 32 and 64 (short iterations) stage X in
    // registers, so the barrier of an iteration waits for LDS writes only and
    // the deeper loads stay in flight; row tiles of 128, and the 16-bit format's
    // of 64, load X straight into LDS one iteration ahead (their registers hold
    // the accumulators and weights).
    // (the 8- and 16-bit formats hold 2 or 4 times the weight registers per
    // tile: the shallowest pipeline)
    constexpr int P = WF != WF_INT4 ? 2 : TM == 1 ? (WN == 2 ? 3 : 4) : (TM == 2 && GT != 0 && WN == 4) ? 3 : 2;
    constexpr int U = P % 2 == 0 ? P : 2 * P;          // unroll: X stage (mod P) and LDS buffer (mod 2) static
    constexpr int XS = XREG ? P : 1;
    u32x4 xr[XS][XL];
    auto xbytes = [&](int kb) __attribute__((always_inline)) {
        return (uint32_t)(kb < kb_hi ? kb : kb_lo) * 128u;
    };
    // DMA variant: the X tile of the iteration that starts at kb into As
    auto load_x_lds = [&](int kb, unsigned char* As) __attribute__((always_inline)) {
        const uint32_t kbytes = xbytes(kb);
#pragma unroll
        for (int i = 0; i < XL; i++)
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(Xb + (xoff[i] + kbytes)),
                                             (__attribute__((address_space(3))) void*)(As + (WN * i + wave) * 1024),
                                             16, 0, 0);
    };
    // register variant: load into stage st, later written to LDS at the place
    // the direct-to-LDS load would fill (lane L: 16 bytes at L * 16)
    auto load_x_reg = [&](int st, int kb) __attribute__((always_inline)) {
        const uint32_t kbytes = xbytes(kb);
#pragma unroll
        for (int i = 0; i < XL; i++)
            xr[XREG ? st : 0][i] = *reinterpret_cast<const u32x4*>(Xb + (xoff[i] + kbytes));
    };
    auto store_x = [&](int st, unsigned char* As) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < XL; i++)
            *reinterpret_cast<u32x4*>(As + (WN * i + wave) * 1024 + lane * 16) = xr[XREG ? st : 0][i];
    };

    // ---- weight ring: group g (slots 4 g .. 4 g + 3) holds the tiles of one
    // iteration, slot 4 g + 2 half + column with the ratios (and zero points)
    // of their groups.  Loads past the range re-read the range's first tile
    // (never used).
    constexpr int NG = XREG ? P : 2;
    constexpr int NQ = 1 << WF;                         // 16-byte quads per lane and tile
    constexpr uint32_t TB = 1024u << WF;                // tile bytes
    const char* const Wb = reinterpret_cast<const char*>(W.qw);
    const uint32_t woff0 = (uint32_t)(wave_on ? nt0 : 0) * (uint32_t)KB * TB + (uint32_t)lane * 16u;
    const uint32_t wcol1 = (uint32_t)KB * TB;
    const char* const Rb = reinterpret_cast<const char*>(W.ratios);
    // FS (INT4, 128-row tiles, SwiGLU and residual epilogues): a weight
    // fragment is multiplied by its group's fp16 scale (4 packed multiplies,
    // which the fragment's 8 MFMAs share) instead of the accumulators by the
    // running ratio at each group boundary (128 multiplies per group); the
    // product (q - z) s is rounded to fp16.  With fewer row tiles a fragment
    // serves fewer MFMAs and the ratio costs less, so those keep it; so does
    // the q/k/v GEMM, whose exact sums decide the bf16 rounding of the
    // cached keys and values.
    constexpr bool FS = WF == WF_INT4 && TM == 4 && EPI != EPI_QKV;
    // RT: ratios in use.  The 8- and 16-bit formats have one scale per column
    // (every ratio 1) and one zero point, read once.
    constexpr bool RT = WF == WF_INT4 && !FS;
    u32x4 rw[4 * NG][NQ];
    float rr[4 * NG][NH];
    f16 rs[4 * NG][NH];
    uint32_t rz[4 * NG][NH];
    auto load_w = [&](int q, int kb) __attribute__((always_inline)) {
        const int kk = kb < kb_hi ? kb : kb_lo;
        const int col = (q & 1) ? col1 : col0;
#pragma unroll
        for (int j = 0; j < NQ; j++)
            rw[q][j] = *reinterpret_cast<const u32x4*>(Wb + (woff0 + ((q & 1) ? wcol1 : 0u) + (uint32_t)kk * TB + 1024u * j));
#pragma unroll
        for (int hh = 0; hh < NH; hh++) {
            const uint32_t gi = (uint32_t)((kk * 64 + 32 * hh) >> W.lgG) * (uint32_t)W.N_dev + (uint32_t)col;
            if constexpr (FS) rs[q][hh] = __builtin_bit_cast(f16, W.scales[gi]);
            else if constexpr (RT) rr[q][hh] = *reinterpret_cast<const float*>(Rb + gi * 4u);
            if constexpr (RT && ZP) rz[q][hh] = (uint32_t)W.zeros[gi];
        }
    };
    // DMA variant: the scale ratio of the first tile of the iteration that
    // starts at kb (both columns), two iterations ahead in a ring of two
    // slots, so the group boundary at the end of an iteration never waits
    // for loads of the same iteration (slot it % 2 holds the ratio of
    // iteration it + 2 from the start of iteration it on).
    float rn[2][2];
    auto load_rn = [&](int slot, int kb) __attribute__((always_inline)) {
        if constexpr (!RT) return;
        const int kk = kb < kb_hi ? kb : kb_lo;
        const uint32_t g0 = (uint32_t)((kk * 64) >> W.lgG) * (uint32_t)W.N_dev;
        rn[slot][0] = *reinterpret_cast<const float*>(Rb + (g0 + (uint32_t)col0) * 4u);
        rn[slot][1] = *reinterpret_cast<const float*>(Rb + (g0 + (uint32_t)col1) * 4u);
    };
    auto load_group = [&](int g, int kb) __attribute__((always_inline)) {
        load_w(4 * g, kb);
        load_w(4 * g + 1, kb);
        load_w(4 * g + 2, kb + 1);
        load_w(4 * g + 3, kb + 1);
    };

    f32x16 acc[TM][2];
#pragma unroll
    for (int i = 0; i < TM; i++) { acc[i][0] = f32x16{}; acc[i][1] = f32x16{}; }
    ZeroOff zo0 = zero_off(8.0f), zo1 = zo0;
    if constexpr (WF == WF_INT8) {
        zo0 = zero_off((float)W.zeros[col0]);
        zo1 = zero_off((float)W.zeros[col1]);
    }
    // A fragment of row tile i, step s, tile half: logical chunk 8 half + 2 s + h
    // of row 32 i + c, stored at chunk ^ (row & 15) (row & 15 == c & 15)
    const uint32_t arow = (uint32_t)c * 256u;

    // the MFMAs of the iteration that starts at kb, on the X tile in As and
    // weight group qb; qn: the group of the next iteration (its first ratio)
    auto compute = [&](int kb, const unsigned char* As, int qb, int qn) __attribute__((always_inline)) {
        f16x8 a[2][TM], b[2][2];
        auto prep = [&](int t, int p) __attribute__((always_inline)) {
            const int half = t >> 2, s = t & 3, q = qb + 2 * half, hh = NH == 2 ? (s >> 1) : 0;
            if (ZP && WF == WF_INT4 && (s == 0 || (NH == 2 && s == 2))) {
                zo0 = zero_off((float)rz[q][hh]);
                zo1 = zero_off((float)rz[q + 1][hh]);
            }
            const uint32_t chunk = (uint32_t)((8 * half + 2 * s + h) ^ (c & 15)) * 16u;
#pragma unroll
            for (int i = 0; i < TM; i++)
                a[p][i] = *reinterpret_cast<const f16x8*>(As + (uint32_t)i * 8192u + arow + chunk);
            if constexpr (WF == WF_INT8) {
                b[p][0] = dequant8_u8(rw[q][s >> 1][2 * (s & 1)], rw[q][s >> 1][2 * (s & 1) + 1], zo0.even);
                b[p][1] = dequant8_u8(rw[q + 1][s >> 1][2 * (s & 1)], rw[q + 1][s >> 1][2 * (s & 1) + 1], zo1.even);
            } else if constexpr (WF == WF_F16) {
                b[p][0] = f16_frag(rw[q][s][0], rw[q][s][1], rw[q][s][2], rw[q][s][3]);
                b[p][1] = f16_frag(rw[q + 1][s][0], rw[q + 1][s][1], rw[q + 1][s][2], rw[q + 1][s][3]);
            } else {
                b[p][0] = dequant8(rw[q][0][s], zo0, dq);
                b[p][1] = dequant8(rw[q + 1][0][s], zo1, dq);
                if constexpr (FS) {
                    const f16 s0 = rs[q][hh], s1 = rs[q + 1][hh];
                    b[p][0] = b[p][0] * f16x8{s0, s0, s0, s0, s0, s0, s0, s0};
                    b[p][1] = b[p][1] * f16x8{s1, s1, s1, s1, s1, s1, s1, s1};
                }
            }
        };
        // After step t, if step t + 1 (step 0 of the next iteration for
        // t = 7) starts a group inside the range, the accumulators take
        // its ratio s_prev / s_new.  Doing it here, interleaved with the
        // last MFMAs of the old group, keeps the multiplies off the
        // boundary between the groups' MFMA streams.
        auto next_group = [](int t) { return t == 7 || (GT <= 1 && t == 3) || (GT == 0 && (t & 1) == 1); };
        prep(0, 0);
#pragma unroll
        for (int t = 0; t < 8; t++) {
            const int p = t & 1;
            if (t + 1 < 8) prep(t + 1, p ^ 1);
#pragma unroll
            for (int i = 0; i < TM; i++) {
                acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[p][i], b[p][0], acc[i][0], 0, 0, 0);
                acc[i][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[p][i], b[p][1], acc[i][1], 0, 0, 0);
            }
            if (RT && next_group(t)) {
                const int tn = (t + 1) & 7;                       // the next step
                const int half = tn >> 2, hh = NH == 2 ? ((tn & 3) >> 1) : 0;
                const int q = (t == 7 ? qn : qb) + 2 * half;
                const int k = (kb + (t == 7 ? 2 : 0) + half) * 64 + (tn & 3) * 16;
                const bool start = k < kb_hi * 64 && (k & Gm1) == 0;
                float r0 = rr[q][hh], r1 = rr[q + 1][hh];
                if (!XREG && t == 7) {          // the next iteration's first tile (NH == 1)
                    r0 = rn[(qb >> 2) ^ 1][0];
                    r1 = rn[(qb >> 2) ^ 1][1];
                }
                const float f0 = start ? r0 : 1.0f, f1 = start ? r1 : 1.0f;
#pragma unroll
                for (int i = 0; i < TM; i++)
#pragma unroll
                    for (int e = 0; e < 16; e++) {
                        acc[i][0][e] *= f0;
                        acc[i][1][e] *= f1;
                    }
                sched_step<TM, TM == 4 ? 16 : 20>();
            } else {
                sched_step<TM, TM == 4 ? 4 : 6>();
            }
        }
    };

    // ---- what the epilogue reads, requested before the main loop: the scale
    // of the range's last group (1 with fragment scales), and where the thread
    // ends with few rows (EARLY) the residual or the RoPE factors of them.
    // At the end each of these costs the block a memory round trip (pos and
    // then cos / sin: two).
    constexpr int NP = 16 * TM / KG;                    // register rows that this thread ends with
    constexpr int NE = NP < 16 ? NP : 16;               // rows per epilogue pass
    constexpr bool EARLY = NP <= 8;
    const int rr0 = kg * NP;                            // the first of them
    auto reg_row = [&](int j) { return m0 + 32 * ((rr0 + j) / 16) + 8 * (((rr0 + j) % 16) / 4) + 4 * h + (rr0 + j) % 4; };
    auto clamp_row = [&](int j) { const int m = reg_row(j); return m < M ? m : M - 1; };
    const int glast = kb_hi > 0 ? ((kb_hi * 64) - 1) >> W.lgG : 0;
    const float sl0 = FS ? 1.0f : (float)__builtin_bit_cast(f16, W.scales[(size_t)glast * W.N_dev + col0]);
    const float sl1 = FS ? 1.0f : (float)__builtin_bit_cast(f16, W.scales[(size_t)glast * W.N_dev + col1]);
    // q/k/v: the column pair (nt0 * 32 + c, + 32) holds dims dim0 and dim1 of
    // head `head` of q (kind 0), k (1) or v (2): a RoPE pair (rope_block)
    int kind = 0, head = 0, dim0 = 0, dim1 = 0;
    if (EPI == EPI_QKV) {
        const int d = ep.head_dim, qd = ep.nq * d, kd = ep.nkv * d;
        int n = (wave_on ? nt0 : 0) * 32;
        if (n >= qd + kd) { kind = 2; n -= qd + kd; }
        else if (n >= qd) { kind = 1; n -= qd; }
        head = n / d;
        const int p0 = (n - head * d) / 32;
        dim0 = 32 * rope_block(p0, d) + c;
        dim1 = 32 * rope_block(p0 + 1, d) + c;
    }
    float e0[NE], e1[NE];                               // residual pair, or cos and sin, of the pass's rows
    auto epi_load = [&](int j0) __attribute__((always_inline)) {
        if (EPI == EPI_RESID) {
#pragma unroll
            for (int e = 0; e < NE; e++) {
                const size_t o = (size_t)clamp_row(j0 + e) * W.N;
                e0[e] = ep.resid[o + col0];
                e1[e] = ep.resid[o + col1];
            }
        } else if (EPI == EPI_QKV) {
            int ps[NE];
#pragma unroll
            for (int e = 0; e < NE; e++) ps[e] = ep.pos[clamp_row(j0 + e)];
#pragma unroll
            for (int e = 0; e < NE; e++) {
                const size_t o = (size_t)ps[e] * (ep.head_dim / 2) + dim0;
                e0[e] = ep.rope_cos[o];
                e1[e] = ep.rope_sin[o];
            }
        }
    };
    if (EARLY) epi_load(0);

    if constexpr (XREG) {
        // iteration it (u = it mod U): X of it + P into stage u mod P (X of it
        // is in LDS already), the MFMAs of it on LDS buffer u mod 2 and weight
        // group u mod P, then the weights of it + P into that group, X of
        // it + 1 into the other LDS buffer, and the barrier.  A k group whose
        // range is shorter than the block's longest only loads, stores and
        // waits in the last iteration.
#pragma unroll
        for (int j = 0; j < P; j++) {
            load_x_reg(j, kb_lo + 2 * j);
            load_group(j, kb_lo + 2 * j);
        }
        store_x(0, As0);
        __syncthreads();
        for (int it0 = 0; it0 < nit; it0 += U) {
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (it0 + u >= nit) break;
                const int kb = kb_lo + 2 * (it0 + u);
                const int st = u % P;
                load_x_reg(st, kb + 2 * P);
                if (kb < kb_hi) compute(kb, (u & 1) ? As1 : As0, 4 * st, 4 * ((u + 1) % P));
                load_group(st, kb + 2 * P);
                store_x((u + 1) % P, (u & 1) ? As0 : As1);
                __syncthreads();
            }
        }
    } else {
        // iteration it: X and weights of it + 1 requested (X straight to LDS),
        // the MFMAs of it, then the barrier, whose workgroup release waits for
        // the block's outstanding loads.  With it == nit (the odd partner of
        // the last iteration) only the loads and the barrier run.
        auto iteration = [&](int it, const unsigned char* As, unsigned char* As_next, int qb, int qn)
            __attribute__((always_inline)) {
            const int kb = kb_lo + 2 * it;
            load_rn(qb >> 2, kb + 4);
            load_x_lds(kb + 2, As_next);
            load_group(qn / 4, kb + 2);
            if (kb < kb_hi) compute(kb, As, qb, qn);
            __syncthreads();
        };
        load_x_lds(kb_lo, As0);
        load_group(0, kb_lo);
        load_rn(1, kb_lo + 2);
        __syncthreads();
        for (int it = 0; it < nit; it += 2) {
            iteration(it, As0, As1, 0, 4);
            iteration(it + 1, As1, As0, 4, 0);
        }
    }

    // ---- the k groups' sums meet in LDS: group q ends with the sums of the
    // register rows q NP .. q NP + NP - 1 (register row r is row m0 + 32 (r / 16)
    // + 8 (r % 16 / 4) + 4 h + r % 4), its own part plus the others' in group order
    float t0[NP], t1[NP];
    if constexpr (KG == 1) {
#pragma unroll
        for (int j = 0; j < NP; j++) {
            t0[j] = acc[j / 16][0][j % 16] * sl0;
            t1[j] = acc[j / 16][1][j % 16] * sl1;
        }
    } else {
        float2* const ex = reinterpret_cast<float2*>(smem);   // [target][writer][WN][NP][64]
        // (the loop's last barrier: every wave has read its X tiles)
#pragma unroll
        for (int q = 0; q < KG; q++) {
            if (kg == q) {
#pragma unroll
                for (int j = 0; j < NP; j++) {
                    t0[j] = acc[(q * NP + j) / 16][0][(q * NP + j) % 16] * sl0;
                    t1[j] = acc[(q * NP + j) / 16][1][(q * NP + j) % 16] * sl1;
                }
            } else {
                const int w = kg < q ? kg : kg - 1;
#pragma unroll
                for (int j = 0; j < NP; j++)
                    ex[(((q * (KG - 1) + w) * WN + wave) * NP + j) * 64 + lane] =
                        float2{acc[(q * NP + j) / 16][0][(q * NP + j) % 16] * sl0,
                               acc[(q * NP + j) / 16][1][(q * NP + j) % 16] * sl1};
            }
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < KG - 1; w++)
#pragma unroll
            for (int j = 0; j < NP; j++) {
                const float2 v = ex[(((kg * (KG - 1) + w) * WN + wave) * NP + j) * 64 + lane];
                t0[j] += v.x;
                t1[j] += v.y;
            }
    }
    // Epilogue of the thread's values j0 .. j0 + NE - 1.  What it reads
    // (epi_load) is requested for all its rows before the first store: a store
    // could alias a later read, so interleaved they would cost a memory round
    // trip per row.
    auto epilogue = [&](int j0) __attribute__((always_inline)) {
        int mr[NE];
#pragma unroll
        for (int e = 0; e < NE; e++) {
            const int m = reg_row(j0 + e);
            mr[e] = m < M ? m : -1;
        }
        if (!EARLY) epi_load(j0);
        if (EPI == EPI_RESID) {
#pragma unroll
            for (int e = 0; e < NE; e++) {
                if (mr[e] < 0) continue;
                const size_t o = (size_t)mr[e] * W.N;
                ep.out_f32[o + col0] = e0[e] + t0[j0 + e];
                ep.out_f32[o + col1] = e1[e] + t1[j0 + e];
            }
        } else if (EPI == EPI_SWIGLU) {
            const int f = (nt0 / 2) * 32 + c;          // tile pair (2j, 2j+1) = gate block j, up block j
            bool bad = false;
#pragma unroll
            for (int e = 0; e < NE; e++)
                if (mr[e] >= 0) ep.act_out[(size_t)mr[e] * ep.F_pad + f] = act_f16(silu(t0[j0 + e]) * t1[j0 + e], bad);
            flag_range(ep.err, bad);
        } else {
#pragma unroll
            for (int e = 0; e < NE; e++) {
                if (mr[e] < 0) continue;
                const float v0 = t0[j0 + e], v1 = t1[j0 + e];
                float o0 = v0, o1 = v1;
                if (kind < 2) {                         // RoPE on q and k
                    o0 = v0 * e0[e] - v1 * e1[e];
                    o1 = v1 * e0[e] + v0 * e1[e];
                }
                const uint16_t b0 = bf16_bits_rne(o0), b1 = bf16_bits_rne(o1);
                uint16_t* dst;
                if (kind == 0) {
                    dst = ep.q_out + ((size_t)mr[e] * ep.nq + head) * ep.head_dim;
                } else {
                    uint16_t* cache = (kind == 1) ? ep.k_cache : ep.v_cache;
                    dst = cache + (size_t)head * ep.cache_stride_h + (size_t)(ep.slot_base + mr[e]) * ep.head_dim;
                }
                dst[dim0] = b0;
                dst[dim1] = b1;
            }
        }
    };

    if (gs.S > 1) {
        // ---- split K: store the partial sums (register row, lane order: 512
        // contiguous bytes per wave and row); the last block of the tile to
        // arrive adds the S partials in range order.  The partials are written
        // and read with device-coherent (relaxed, agent scope) accesses, which
        // go past the non-coherent per-XCD L2, so the count only has to follow
        // their completion: no cache write-back or invalidation is needed.
        const size_t tile = (size_t)(rb * gs.ncb + cb);
        constexpr size_t TP = (size_t)TM * 16 * WN * 64;      // pairs of one tile
        unsigned long long* const mine = gs.part + (tile * gs.S + sp) * TP + (size_t)(rr0 * WN + wave) * 64 + lane;
#pragma unroll
        for (int j = 0; j < NP; j++)
            __hip_atomic_store(mine + (size_t)j * WN * 64,
                               (unsigned long long)__float_as_uint(t1[j]) << 32 | __float_as_uint(t0[j]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's partial stores are complete
        __syncthreads();
        if (tid == 0)
            last_flag = __hip_atomic_fetch_add(gs.cnt + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
                        (unsigned)gs.S;
        __syncthreads();
        if (!last_flag) return;
        // The sum, NB register rows at a time: the values of SB ranges are
        // requested together (one memory round trip); with two ranges only the
        // other one's.
        constexpr int NB = NP < 16 ? NP : 16, SB = 32 / NB;
#pragma unroll
        for (int j0 = 0; j0 < NP; j0 += NB) {
            if (gs.S == 2) {
                const unsigned long long* src = gs.part + (tile * 2 + (1 - sp)) * TP + (size_t)((rr0 + j0) * WN + wave) * 64 + lane;
                unsigned long long v[NB];
#pragma unroll
                for (int j = 0; j < NB; j++)
                    v[j] = __hip_atomic_load(src + (size_t)j * WN * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int j = 0; j < NB; j++) {
                    t0[j0 + j] += __uint_as_float((unsigned)v[j]);
                    t1[j0 + j] += __uint_as_float((unsigned)(v[j] >> 32));
                }
                continue;
            }
            float a0[NB], a1[NB];
#pragma unroll
            for (int j = 0; j < NB; j++) { a0[j] = 0.f; a1[j] = 0.f; }
            for (int s0 = 0; s0 < gs.S; s0 += SB) {
                unsigned long long v[SB][NB];
#pragma unroll
                for (int s = 0; s < SB; s++) {
                    const int ss = s0 + s < gs.S ? s0 + s : gs.S - 1;
                    const unsigned long long* src = gs.part + (tile * gs.S + ss) * TP + (size_t)((rr0 + j0) * WN + wave) * 64 + lane;
#pragma unroll
                    for (int j = 0; j < NB; j++)
                        v[s][j] = __hip_atomic_load(src + (size_t)j * WN * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int s = 0; s < SB; s++)
                    if (s0 + s < gs.S) {
#pragma unroll
                        for (int j = 0; j < NB; j++) {
                            a0[j] += __uint_as_float((unsigned)v[s][j]);
                            a1[j] += __uint_as_float((unsigned)(v[s][j] >> 32));
                        }
                    }
            }
#pragma unroll
            for (int j = 0; j < NB; j++) { t0[j0 + j] = a0[j]; t1[j0 + j] = a1[j]; }
        }
    }
    if (!wave_on) return;
#pragma unroll
    for (int j0 = 0; j0 < NP; j0 += NE) epilogue(j0);
}

template <int EPI, int TM, int GT, bool ZP, int WF, int WN, int KG>
int launch_v(const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmShape& gs, hipStream_t stream) {
    const int blocks = gs.nrb * gs.ncb * gs.S;
    const size_t lds = lds_bytes<TM, WN, KG>();
    static LdsLimit lim;
    if (ensure_lds_limit(lim, (const void*)gemm_w4_kernel<EPI, TM, GT, ZP, WF, WN, KG>, lds)) return -1;
    hipLaunchKernelGGL((gemm_w4_kernel<EPI, TM, GT, ZP, WF, WN, KG>), dim3(blocks), dim3(64 * WN * KG), lds, stream, X,
                       ldx, W, ep, gs);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// the block shapes of one row tile: 256 or 128 columns, k groups
template <int EPI, int TM, int GT, bool ZP, int WF>
int launch_shape(const GemmPlan& p, const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmShape& gs,
                 hipStream_t stream) {
    if constexpr (TM == 4 || (TM == 2 && WF == WF_F16)) {
        return launch_v<EPI, TM, GT, ZP, WF, 4, 1>(X, ldx, W, ep, gs, stream);
    } else {
        if (p.WN == 4 && p.KG == 1) return launch_v<EPI, TM, GT, ZP, WF, 4, 1>(X, ldx, W, ep, gs, stream);
        if (p.WN == 4 && p.KG == 2) return launch_v<EPI, TM, GT, ZP, WF, 4, 2>(X, ldx, W, ep, gs, stream);
        if constexpr (!(TM == 2 && GT == 0 && ZP))
            if (p.WN == 2 && p.KG == 4) return launch_v<EPI, TM, GT, ZP, WF, 2, 4>(X, ldx, W, ep, gs, stream);
        return -1;
    }
}

// row tiles of 128 only for 4-bit weights in groups of 64 or more without zero
// points (with them, and for the 8-bit format, they were built and measured: at
// 200 to 800 rows slower than row tiles of 64 in all but one product)
template <int EPI, int GT, bool ZP, int WF>
int launch_tm(const GemmPlan& p, const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmShape& gs,
              hipStream_t stream) {
    if (p.TM == 1) return launch_shape<EPI, 1, GT, ZP, WF>(p, X, ldx, W, ep, gs, stream);
    if (p.TM == 2) return launch_shape<EPI, 2, GT, ZP, WF>(p, X, ldx, W, ep, gs, stream);
    if constexpr (WF == WF_INT4 && !ZP && GT != 0)
        if (p.TM == 4) return launch_shape<EPI, 4, GT, ZP, WF>(p, X, ldx, W, ep, gs, stream);
    return -1;
}

template <int EPI>
int launch_epi(const GemmPlan& p, const f16* X, int ldx, const DevLinear& W, const EpiArgs& ep, const GemmShape& gs,
               hipStream_t stream) {
    const bool zp = W.zeros != nullptr;
    const int gt = W.lgG == 5 ? 0 : W.lgG == 6 ? 1 : 2;
    // 8-bit: zero points, groups of 128; 16-bit: neither
    if (W.wf == WF_INT8) return zp && gt == 2 ? launch_tm<EPI, 2, true, WF_INT8>(p, X, ldx, W, ep, gs, stream) : -1;
    if (W.wf == WF_F16) return !zp && gt == 2 ? launch_tm<EPI, 2, false, WF_F16>(p, X, ldx, W, ep, gs, stream) : -1;
    if (zp) {
        if (gt == 0) return launch_tm<EPI, 0, true, WF_INT4>(p, X, ldx, W, ep, gs, stream);
        if (gt == 1) return launch_tm<EPI, 1, true, WF_INT4>(p, X, ldx, W, ep, gs, stream);
        return launch_tm<EPI, 2, true, WF_INT4>(p, X, ldx, W, ep, gs, stream);
    }
    if (gt == 0) return launch_tm<EPI, 0, false, WF_INT4>(p, X, ldx, W, ep, gs, stream);
    if (gt == 1) return launch_tm<EPI, 1, false, WF_INT4>(p, X, ldx, W, ep, gs, stream);
    return launch_tm<EPI, 2, false, WF_INT4>(p, X, ldx, W, ep, gs, stream);
}

}  // namespace
