// W4A16 GEMV for the decode stage, one kernel per linear (B <= 8 rows):
// y[b][n] = sum_k x[b][k] W[k][n].  The INT8 and F16 weight formats go
// through the same kernel with their own fragment unpack (gemv_core.h).
//
// Block: NW waves on CT column tiles (a pair, 64 device columns: a RoPE pair of
// q/k blocks, a gate/up pair, or two residual tiles; or one residual tile) and
// the block's k range; the waves split the k range evenly and each streams the
// tiles of its share through a register ring.  The two tiles of a pair share
// the activation fragments and are two independent MFMA chains.  The wave partials meet in
// LDS in a fixed order.  Grid: (N_dev / 64, ksplit); with ksplit > 1 the
// residual epilogue adds into an output that an earlier launch cleared (the
// blocks of the first k range add the residual as well).
//
// A launch is short (a few microseconds), so what counts is the number of
// dependent memory round trips.  The activations are requested first, then the
// first weight tiles: a wave's loads return in order, so the rows can be
// prepared (and, with NORM, normalised) while the weights are on their way.
// A wave prepares just the k range it works on, so it starts without a barrier
// (NORM: one, for the row sums), the rows stay in registers from the load to
// the prepared form (gemv_core.h), and what the epilogue reads (positions and
// RoPE factors, residual) is requested before the main loop.
//
// Per launch, before (block-wide passes through LDS, weights requested first,
// one tile at a time) / now: Llama-8B q/k/v 13.2 / 9.3 us, o_proj 8.5 / 6.0,
// gate/up 18.8 / 15.5, down 11.9 / 9.1 (5 rows, kernel trace).
//
// NORM: the rows are fp32 and every block normalises them (RMSNorm, rounded to
// bf16), in registers: the caller uses it where they fit (gemv_norm_fits);
// larger batches are normalised once by a launch of their own.
#include "common.h"
#include "gemv_core.h"
#include "launch.h"

namespace {

constexpr int MAXB = 8;
constexpr int NX = 4;            // 8-element activation chunks a thread holds
constexpr int kRawBuffer = 0x00020000;       // buffer descriptor word 3: raw 32-bit data, stride 0

// WF: weight format (WeightFormat); the 8-bit format always has zero points (ZP)
template <int EPI, bool NORM, bool ZP, bool G32, int WF, int NW, int CT>
__global__ void __launch_bounds__(NW * 64) gemv_w4_kernel(GemvArgs a) {
    constexpr int NT = NW * 64;
    constexpr int NQ = 1 << WF;                  // 16-byte quads per lane and tile
    constexpr int RD = (8 / CT >> WF) ? (8 / CT >> WF) : 1;   // steps (CT tiles) in flight per wave: 8 KB
    static_assert(CT == 2 || EPI == EPI_RESID, "q/k/v and gate/up work on tile pairs");
    constexpr bool UV = ZP && !G32;              // correction per 64-k tile with a zero point (else z = 8: c64)
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const DevLinear& W = a.W;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.x * CT;              // first column tile
    const int KB = W.K_pad / 64;
    const int kb_lo = (int)((long long)blockIdx.y * KB / a.ksplit);
    const int kb_hi = (int)((long long)(blockIdx.y + 1) * KB / a.ksplit);
    const int klo = kb_lo * 64, klen = (kb_hi - kb_lo) * 64;
    const int ldx = klen + 8;
    const int B = a.B;
    const int nkb = kb_hi - kb_lo;
    f16* xs = reinterpret_cast<f16*>(smem);                                   // [B][ldx]
    f16* zero = reinterpret_cast<f16*>(smem + B * ldx * 2);                   // [64]
    // corrections per 64-k tile (z = 8: one float; UV: a pair), with groups
    // of 32 pairs per 32-k segment (gemv_core.h)
    float* c64 = reinterpret_cast<float*>(zero + 64);                         // [nkb][GEMV_ROWS]
    float2* uv = reinterpret_cast<float2*>(c64);                              // [nkb or 2 nkb][GEMV_ROWS]
    float* ssq = c64 + nkb * GEMV_ROWS * (G32 ? 4 : UV ? 2 : 1);              // [B][nkb] (NORM)
    float* red = reinterpret_cast<float*>(smem + a.off_red);                  // [NW][CT][B][32], over the rows if 0
    const int ka = kb_lo + wave * nkb / NW, kz = kb_lo + (wave + 1) * nkb / NW;   // this wave's k tiles

    // ---- what the epilogue reads (wave b handles row b, lane = column of the
    // pair), requested first: everything after it is on its way when it lands
    const int eb = wave < B ? wave : 0;
    const int ecol = t0 * 32 + lane % (32 * CT);
    float e0 = 0.f, e1 = 0.f;
    int pos = 0, slot = 0, kind = 0, head = 0, dim = 0;
    if constexpr (EPI == EPI_QKV) {
        pos = a.ep.pos[eb];
        slot = a.ep.slot_dev ? a.ep.slot_dev[eb] : a.ep.slot_base + eb;
    } else if constexpr (EPI == EPI_RESID) {
        if (blockIdx.y == 0 && a.ep.resid) e0 = a.ep.resid[(size_t)eb * W.N + ecol];
    }

    // ---- this wave's activations: chunk i is row i / nc, elements 8 (i % nc) .. + 7
    // of the k range the wave works on, so no wave waits for another's
    const int nc = (kz - ka) * 8, total = B * nc, kw = ka * 64;
    struct Chunk { u32x4 w0, w1, g; };            // fp16 values in w0; NORM: fp32 in w0, w1, gamma in g
    Chunk x[NX];
    auto row_of = [&](int i) { return i < total ? i / nc : 0; };
    auto load_chunk = [&](Chunk& ch, int i) __attribute__((always_inline)) {
        const int b = row_of(i), c = i < total ? i - b * nc : 0;
        if constexpr (NORM) {
            const uint32_t* p = reinterpret_cast<const uint32_t*>(a.x_f32 + (size_t)b * W.K + kw + 8 * c);
            ch.w0 = *reinterpret_cast<const u32x4*>(p);
            ch.w1 = *reinterpret_cast<const u32x4*>(p + 4);
            ch.g = *reinterpret_cast<const u32x4*>(a.gamma + kw + 8 * c);
        } else {
            ch.w0 = *reinterpret_cast<const u32x4*>(a.x_f16 + (size_t)b * a.ldx + kw + 8 * c);
        }
    };
#pragma unroll
    for (int j = 0; j < NX; j++)
        if (j * 64 < total) load_chunk(x[j], lane + j * 64);     // (uniform)

    // ---- the wave's first RD steps of weight tiles
    u32x4 w[RD][CT][NQ];
    uint32_t sa[RD][CT], sb[RD][CT];
    // Loads past the end of the run are issued all the same (a load under a
    // branch would cost the loop a wait for every load in flight), at an offset
    // past the end of the buffer: they return 0 and move no data.  (Re-reading
    // the run's first tile instead: INT8 Qwen-7B, 5 rows, 78.0 against 73.3 us a
    // layer, INT4 within 1%.)
    const uint32_t ngp = (uint32_t)W.KG * (uint32_t)W.N_dev;
    const GemvRun wr = gemv_run_bytes(t0, CT, W.K_pad, WF);
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(W.qw) + wr.first / 4, 0, (int)wr.bytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(
        ZP ? (void*)const_cast<uint32_t*>(W.sz) : (void*)const_cast<uint16_t*>(W.scales), 0, (int)(ngp * (ZP ? 4u : 2u)),
        kRawBuffer);
    auto load_param = [&](uint32_t off) __attribute__((always_inline)) -> uint32_t {
        if constexpr (ZP) return __builtin_amdgcn_raw_buffer_load_b32(grs, off, 0, 0);
        else return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(grs, off, 0, 0);
    };
    constexpr uint32_t GS = ZP ? 4u : 2u;
    const uint32_t lw = (uint32_t)lane * 16u, lg = (uint32_t)(lane & 31) * GS;
    auto load_pair = [&](int u, int kb) __attribute__((always_inline)) {
        const uint32_t grow = (((uint32_t)kb * 64u) >> W.lgG) * (uint32_t)W.N_dev;
#pragma unroll
        for (int t = 0; t < CT; t++) {
            const uint32_t wo = kb < kz ? (uint32_t)(t * KB + kb) << (10 + WF) : kGemvPastEnd;
            const uint32_t go = kb < kz ? (grow + (uint32_t)(t0 + t) * 32u) * GS : kGemvPastEnd;
#pragma unroll
            for (int j = 0; j < NQ; j++) w[u][t][j] = __builtin_amdgcn_raw_buffer_load_b128(wrs, wo + lw + 1024u * j, 0, 0);
            if (WF != WF_F16) sa[u][t] = load_param(go + lg);
            if (G32) sb[u][t] = load_param(go + lg + (kb < kz ? (uint32_t)W.N_dev * GS : 0u));
        }
    };
    // (slot by slot, so that the wait for a slot leaves the later ones in flight,
    // in the loop too)
#pragma unroll
    for (int u = 0; u < RD; u++) {
        __builtin_amdgcn_sched_barrier(0);
        load_pair(u, ka + u);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EPI == EPI_QKV) {
        const int d = a.ep.head_dim, qd = a.ep.nq * d, kd = a.ep.nkv * d;
        int nn = t0 * 32;
        if (nn >= qd + kd) { kind = 2; nn -= qd + kd; }
        else if (nn >= qd) { kind = 1; nn -= qd; }
        head = nn / d;
        const int p0 = (nn - head * d) / 32;
        // the pair's tiles hold dims dim0 (lanes below 32) and their RoPE partners
        const int dim0 = 32 * rope_block(p0, d) + (lane & 31);
        dim = lane < 32 ? dim0 : 32 * rope_block(p0 + 1, d) + (lane & 31);
        const size_t rope = (size_t)pos * (d / 2) + dim0;
        e0 = a.ep.rope_cos[rope];
        e1 = a.ep.rope_sin[rope];
    }

    // ---- the rows, prepared (gemv_core.h), into LDS
    if (lane < 8) reinterpret_cast<u32x4*>(zero)[lane] = u32x4{0u, 0u, 0u, 0u};    // (every wave: the same values)
    const f16x2 sixteenth = f16x2{(f16)0.0625f, (f16)0.0625f};
    // words of fp16 pairs (0,1) (2,3) (4,5) (6,7) of chunk i; the 8 chunks of
    // a 64-k tile sit in 8 adjacent lanes, which meet with DPP row operations
    auto prepare = [&](int i, uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) __attribute__((always_inline)) {
        const bool ok = i < total;
        const int b = row_of(i), c = (ka - kb_lo) * 8 + (ok ? i - b * nc : 0);      // (within the block's range)
        const f16x2 x0 = __builtin_bit_cast(f16x2, w0), x2 = __builtin_bit_cast(f16x2, w2);
        const f16x2 x1 = __builtin_bit_cast(f16x2, w1) * sixteenth, x3 = __builtin_bit_cast(f16x2, w3) * sixteenth;
        float e = ((float)x0[0] + (float)x0[1]) + ((float)x2[0] + (float)x2[1]);
        float o = ((float)x1[0] + (float)x1[1]) + ((float)x3[0] + (float)x3[1]);
        if (ok)
            *reinterpret_cast<u32x4*>(xs + b * ldx + 8 * c) =
                u32x4{w0, __builtin_bit_cast(uint32_t, x1), w2, __builtin_bit_cast(uint32_t, x3)};
        e += dpp_mov<0xB1>(e);
        o += dpp_mov<0xB1>(o);
        e += dpp_mov<0x4E>(e);
        o += dpp_mov<0x4E>(o);
        if (G32 && ok && (c & 3) == 0) uv[(c >> 2) * GEMV_ROWS + b] = float2{e + o, e + 16.0f * o};
        if (!G32) {
            e += dpp_mov<0x141>(e);
            o += dpp_mov<0x141>(o);
            if (ok && (c & 7) == 0) {
                if (UV) uv[(c >> 3) * GEMV_ROWS + b] = float2{e + o, e + 16.0f * o};
                else c64[(c >> 3) * GEMV_ROWS + b] = gemv_c64(e, o);
            }
        }
    };
    if constexpr (NORM) {
        // sums of squares per row and 64-k tile; after the barrier every wave
        // adds them up for itself, 8 lanes to a row
#pragma unroll
        for (int j = 0; j < NX; j++) {
            if (j * 64 >= total) break;
            const int i = lane + j * 64, b = row_of(i);
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t u0 = x[j].w0[e], u1 = x[j].w1[e];
                const float v0 = __uint_as_float(u0), v1 = __uint_as_float(u1);
                ss += v0 * v0 + v1 * v1;
            }
            ss = row_sum<8>(ss);
            if (i < total && (i & 7) == 0) ssq[b * nkb + (ka - kb_lo) + ((i - b * nc) >> 3)] = ss;
        }
        __syncthreads();
        float t = 0.f;
        const int rb = min(lane >> 3, B - 1);
        for (int i = lane & 7; i < nkb; i += 8) t += ssq[rb * nkb + i];
        const float rinv = 1.0f / sqrtf(row_sum<8>(t) / (float)W.K + a.eps);
        bool bad = false;
#pragma unroll
        for (int j = 0; j < NX; j++) {
            if (j * 64 >= total) break;
            const int i = lane + j * 64;
            const float rr = __shfl(rinv, row_of(i) * 8, 64);
            uint32_t q[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {                       // elements 2 e, 2 e + 1
                const uint32_t u0 = e < 2 ? x[j].w0[2 * e] : x[j].w1[2 * e - 4];
                const uint32_t u1 = e < 2 ? x[j].w0[2 * e + 1] : x[j].w1[2 * e - 3];
                const uint32_t gg = x[j].g[e];
                const f16 h0 = act_f16(__uint_as_float(u0) * rr * __uint_as_float(gg << 16), bad);
                const f16 h1 = act_f16(__uint_as_float(u1) * rr * __uint_as_float(gg & 0xFFFF0000u), bad);
                q[e] = (uint32_t)__builtin_bit_cast(uint16_t, h0) | (uint32_t)__builtin_bit_cast(uint16_t, h1) << 16;
            }
            prepare(i, q[0], q[1], q[2], q[3]);
        }
        flag_range(a.ep.err, bad);
    } else {
#pragma unroll
        for (int j = 0; j < NX; j++) {
            if (j * 64 >= total) break;
            prepare(lane + j * 64, x[j].w0[0], x[j].w0[1], x[j].w0[2], x[j].w0[3]);
        }
        for (int i0 = NX * 64; i0 < total; i0 += NX * 64) {     // long ranges of many rows
#pragma unroll
            for (int j = 0; j < NX; j++) load_chunk(x[j], i0 + lane + j * 64);
#pragma unroll
            for (int j = 0; j < NX; j++) prepare(i0 + lane + j * 64, x[j].w0[0], x[j].w0[1], x[j].w0[2], x[j].w0[3]);
        }
    }
    // (a wave reads only what it wrote itself, and its LDS operations are
    // served in order)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // ---- main loop: partial sums of this wave's two tiles, kept in registers.
    // The A operand of this lane (gemv_core.h): MFMA row m = lane % 16 (batch
    // row bm, column half cm), k block lane / 16 (column half c1, k half h)
    const int h = lane >> 5, c = lane & 31;
    const DqConst dq = dq_const();
    const int am = lane & 15, cm = (am >> 2) & 1, bm = 4 * (am >> 3) + (am & 3), c1 = (lane >> 4) & 1;
    const bool valid = cm == c1 && bm < B;
    const f16* abase = (valid ? xs + bm * ldx : zero) + 8 * h;
    const int astride = valid ? 64 : 0;
    const f32x4_t fz = {0.f, 0.f, 0.f, 0.f};
    float p[CT][4] = {};
    for (int k0 = ka; k0 < kz; k0 += RD) {
#pragma unroll
        for (int u = 0; u < RD; u++) {
            const int kb = k0 + u;
            if (kb < kz) {                                      // wave-uniform
                const int kr = kb - kb_lo;
                const f16* xk = abase + kr * astride;
                f16x8 ax[4];
#pragma unroll
                for (int s = 0; s < 4; s++) ax[s] = *reinterpret_cast<const f16x8*>(xk + 16 * s);
                f32x4_t acc[CT];
#pragma unroll
                for (int t = 0; t < CT; t++) acc[t] = fz;
                if constexpr (G32) {                            // k 0..31 and k 32..63 are two groups
#pragma unroll
                    for (int hf = 0; hf < 2; hf++) {
#pragma unroll
                        for (int t = 0; t < CT; t++) {
                            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ax[2 * hf], dequant8_raw(w[u][t][0][2 * hf], dq), fz, 0, 0, 0);
                            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ax[2 * hf + 1], dequant8_raw(w[u][t][0][2 * hf + 1], dq), acc[t], 0, 0, 0);
                        }
                        const float2* cr = uv + (2 * kr + hf) * GEMV_ROWS + 4 * h;
#pragma unroll
                        for (int t = 0; t < CT; t++) {
                            const uint32_t sw = hf ? sb[u][t] : sa[u][t];
                            const float sc = gscale(sw), z = gzero<ZP>(sw);
#pragma unroll
                            for (int r = 0; r < 4; r++)
                                p[t][r] = __builtin_fmaf(sc, acc[t][r] - __builtin_fmaf(z, cr[r].y, 1024.0f * cr[r].x), p[t][r]);
                        }
                    }
                } else {
#pragma unroll
                    for (int s = 0; s < 4; s++)
#pragma unroll
                        for (int t = 0; t < CT; t++) {
                            f16x8 bf;
                            if constexpr (WF == WF_INT8) bf = dequant8_u8_raw(w[u][t][s >> 1][2 * (s & 1)], w[u][t][s >> 1][2 * (s & 1) + 1]);
                            else if constexpr (WF == WF_F16) bf = __builtin_bit_cast(f16x8, w[u][t][s]);
                            else bf = dequant8_raw(w[u][t][0][s], dq);
                            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ax[s], bf, acc[t], 0, 0, 0);
                        }
                    if constexpr (WF == WF_F16) {
#pragma unroll
                        for (int t = 0; t < CT; t++)
#pragma unroll
                            for (int r = 0; r < 4; r++) p[t][r] += acc[t][r];
                    } else if constexpr (UV) {
                        const float2* cr = uv + kr * GEMV_ROWS + 4 * h;
#pragma unroll
                        for (int t = 0; t < CT; t++) {
                            const float sc = gscale(sa[u][t]), z = gzero<true>(sa[u][t]);
#pragma unroll
                            for (int r = 0; r < 4; r++) {
                                const float co = WF == WF_INT8 ? (1024.0f + z) * cr[r].y
                                                               : __builtin_fmaf(z, cr[r].y, 1024.0f * cr[r].x);
                                p[t][r] = __builtin_fmaf(sc, acc[t][r] - co, p[t][r]);
                            }
                        }
                    } else {
                        const f32x4_t cc = *reinterpret_cast<const f32x4_t*>(c64 + kr * GEMV_ROWS + 4 * h);
#pragma unroll
                        for (int t = 0; t < CT; t++) {
                            const float sc = gscale(sa[u][t]);
#pragma unroll
                            for (int r = 0; r < 4; r++) p[t][r] = __builtin_fmaf(sc, acc[t][r] - cc[r], p[t][r]);
                        }
                    }
                }
            }
            load_pair(u, kb + RD);                              // every step refills its slot, so no load sits
                                                                // under a branch
        }
    }
    if (a.off_red == 0) __syncthreads();   // every wave is done with the activation rows
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const int b = 4 * h + r;
        if (b < B) {
#pragma unroll
            for (int t = 0; t < CT; t++) red[((wave * CT + t) * B + b) * 32 + c] = p[t][r];
        }
    }
    __syncthreads();
    // words for later launches (stores only: nothing waits for them)
    const int blk = blockIdx.y * gridDim.x + blockIdx.x;
    for (int i = blk * NT + tid; i < a.nclear; i += gridDim.x * gridDim.y * NT) a.clear[i] = 0.f;
    if (blk == 0)
        for (int i = tid; i < a.nzero; i += NT) a.zero[i] = 0u;
    if (wave >= B || lane >= 32 * CT) return;

    // ---- epilogue: row eb = wave, column ecol
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < NW; i++) v += red[((i * CT + h) * B + eb) * 32 + c];
    if constexpr (EPI == EPI_RESID) {
        float* o = a.ep.out_f32 + (size_t)eb * W.N + ecol;
        if (a.ksplit == 1) *o = e0 + v;
        else atomicAdd(o, e0 + v);
        return;
    }
    const float other = __shfl_xor(v, 32, 64);
    if constexpr (EPI == EPI_SWIGLU) {
        if (lane < 32) {                                        // gate here, up in the partner
            bool bad = false;
            a.ep.act_out[(size_t)eb * a.ep.F_pad + t0 * 16 + lane] = act_f16(silu(v) * other, bad);
            flag_range(a.ep.err, bad);
        }
    } else {
        float r = v;
        if (kind < 2) r = lane < 32 ? v * e0 - other * e1 : v * e0 + other * e1;     // RoPE on q and k
        uint16_t* dst;
        if (kind == 0) {
            dst = a.ep.q_out + ((size_t)eb * a.ep.nq + head) * a.ep.head_dim;
        } else {
            uint16_t* cache = kind == 1 ? a.ep.k_cache : a.ep.v_cache;
            dst = cache + (size_t)eb * a.ep.cache_stride_b + (size_t)head * a.ep.cache_stride_h + (size_t)slot * a.ep.head_dim;
        }
        dst[dim] = bf16_bits_rne(r);
    }
}

constexpr size_t kLdsMax = 160 * 1024;

// LDS of a block: rows, zero operand, corrections, sums of squares; the wave
// partials after them (a barrier less) unless only over the rows do two blocks
// fit a CU (off_red 0)
size_t lds_bytes(bool norm, bool zp, bool g32, int nw, int ct, int B, int K_pad, int ksplit, int& off_red) {
    const int nkb = (K_pad / 64 + ksplit - 1) / ksplit;
    const size_t rows = (size_t)B * (nkb * 64 + 8) * 2 + 128 + (size_t)nkb * GEMV_ROWS * (g32 ? 16 : zp ? 8 : 4) +
                        (norm ? (size_t)B * nkb * 4 : 0);
    const size_t red = (size_t)nw * ct * B * 32 * 4;
    off_red = rows + red > 80 * 1024 ? 0 : (int)((rows + 15) / 16 * 16);
    return off_red ? off_red + red : std::max(rows, red);
}

template <int EPI, bool NORM, bool ZP, bool G32, int WF, int NW, int CT>
int launch_nw(const GemvArgs& a, hipStream_t stream) {
    const int KB = a.W.K_pad / 64;
    GemvArgs b = a;
    const size_t smem = lds_bytes(NORM, ZP, G32, NW, CT, a.B, a.W.K_pad, a.ksplit, b.off_red);
    if (smem > kLdsMax) return -1;
    if (NORM && (a.ksplit > 1 || a.B * ((KB + NW - 1) / NW) > NX * 8)) return -1;
    static LdsLimit lim;
    if (ensure_lds_limit(lim, (const void*)gemv_w4_kernel<EPI, NORM, ZP, G32, WF, NW, CT>, smem)) return -1;
    dim3 grid(a.W.N_dev / (32 * CT), a.ksplit);
    hipLaunchKernelGGL((gemv_w4_kernel<EPI, NORM, ZP, G32, WF, NW, CT>), grid, dim3(NW * 64), smem, stream, b);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// 8 waves on a tile pair; where that leaves fewer blocks than CUs, 16 waves.
// Residual products in their ordered form (gemv_resid_plan), which only layers
// that the persistent launch could serve take: 16 waves on one tile.
template <int EPI, bool NORM, bool ZP, bool G32, int WF>
int launch_t(const GemvArgs& a, hipStream_t stream) {
    if constexpr (EPI == EPI_RESID) {
        if constexpr (WF == WF_INT4 && !ZP && !G32) {
            if (a.ct == 1) return launch_nw<EPI, NORM, ZP, G32, WF, 16, 1>(a, stream);
        }
        if (a.ct != 2) return -1;
    } else {
        if (a.W.N_dev / 64 <= a.num_cus) return launch_nw<EPI, NORM, ZP, G32, WF, 16, 2>(a, stream);
    }
    return launch_nw<EPI, NORM, ZP, G32, WF, 8, 2>(a, stream);
}

template <bool ZP, bool G32, int WF = WF_INT4>
int launch_zp(int epi, bool norm, const GemvArgs& a, hipStream_t stream) {
    if (epi == EPI_QKV)
        return norm ? launch_t<EPI_QKV, true, ZP, G32, WF>(a, stream) : launch_t<EPI_QKV, false, ZP, G32, WF>(a, stream);
    if (epi == EPI_SWIGLU)
        return norm ? launch_t<EPI_SWIGLU, true, ZP, G32, WF>(a, stream)
                    : launch_t<EPI_SWIGLU, false, ZP, G32, WF>(a, stream);
    if (epi == EPI_RESID && !norm) return launch_t<EPI_RESID, false, ZP, G32, WF>(a, stream);
    return -1;
}

}  // namespace

// Blocks of tile pairs, cut along k until there are two per CU (8 waves each)
// or a wave would be left without a k tile; the ranges meet in the output by
// atomic adds, in any order.  `ordered`: the result must not depend on timing,
// so at most two ranges (adds onto 0 commute); 16 waves on one tile then keep
// the CUs busy, at 1 to 3 us more per layer (Llama-8B, one row, 300 keys:
// 45.4 against 44.5 us; Qwen-0.5B 31.2 against 28.3).  More ranges until the
// activation rows of one (at most 128 KB) and their corrections fit the LDS.
void gemv_resid_plan(GemvArgs& a, bool ordered) {
    const int KB = a.W.K_pad / 64, pairs = a.W.N_dev / 64;
    const bool zp = a.W.sz != nullptr, g32 = a.W.lgG == 5;
    a.ct = ordered ? 1 : 2;
    int ks = ordered ? (2 * pairs < a.num_cus && KB >= 32 ? 2 : 1)
                     : std::max(1, std::min((KB + 7) / 8, 2 * a.num_cus / pairs));
    int off_red;
    while (ks < KB && ((long long)a.B * ((KB + ks - 1) / ks) * 64 * 2 > 128 * 1024 ||
                       lds_bytes(false, zp, g32, a.ct == 1 ? 16 : 8, a.ct, a.B, a.W.K_pad, ks, off_red) > kLdsMax))
        ks++;
    a.ksplit = ks;
}

// (for the host tests: the k ranges and LDS bytes of a residual GEMV)
extern "C" void w4_gemv_resid_plan(int B, int K_pad, int N_dev, int zp, int lgG, int ordered, int num_cus, int* ksplit,
                                   uint64_t* lds) {
    static const uint32_t word = 0;
    GemvArgs a{};
    a.B = B;
    a.num_cus = num_cus;
    a.W.K_pad = K_pad;
    a.W.N_dev = N_dev;
    a.W.lgG = lgG;
    a.W.sz = zp ? &word : nullptr;
    gemv_resid_plan(a, ordered != 0);
    int off_red;
    *ksplit = a.ksplit;
    *lds = lds_bytes(false, zp != 0, lgG == 5, a.ct == 1 ? 16 : 8, a.ct, B, K_pad, a.ksplit, off_red);
}

bool gemv_norm_fits(int B, int K) { return B * ((K / 64 + 7) / 8) <= NX * 8; }

// (for the host tests)
extern "C" void w4_gemv_run_bytes(int tile, int ct, int K_pad, int wf, uint64_t* first, uint32_t* bytes) {
    const GemvRun r = gemv_run_bytes(tile, ct, K_pad, wf);
    *first = r.first;
    *bytes = r.bytes;
}

int launch_gemv_w4(int epi, bool norm, const GemvArgs& a, hipStream_t stream) {
    if (a.B < 1 || a.B > MAXB) return -1;
    if (a.W.wf == WF_INT8) return a.W.sz ? launch_zp<true, false, WF_INT8>(epi, norm, a, stream) : -1;
    if (a.W.wf == WF_F16) return launch_zp<false, false, WF_F16>(epi, norm, a, stream);
    const bool g32 = a.W.lgG == 5;
    if (a.W.sz) return g32 ? launch_zp<true, true>(epi, norm, a, stream) : launch_zp<true, false>(epi, norm, a, stream);
    return g32 ? launch_zp<false, true>(epi, norm, a, stream) : launch_zp<false, false>(epi, norm, a, stream);
}

int load_gemv_w4() { return load_code((const void*)gemv_w4_kernel<EPI_QKV, true, false, false, WF_INT4, 8, 2>); }
