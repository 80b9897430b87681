// Grouped-query causal attention (top.FAttention, Sec. 2.2) for the three
// stages.
//
// Prefill / prefill_kv: flash attention on the 32x32x16 bf16 MFMA.  A block
// works on one kv head, one tile of 32 queries and one chunk of the keys
// those queries see; its waves are the query heads of the kv head's group
// (one head per wave), so every K/V tile staged in LDS serves all of them.
// Chunks split long key ranges across blocks (a causal prefill's late query
// tiles, a prefill_kv over a long history) where the grid would leave CUs idle
// (attn_prefill_plan); work items are ordered longest first.
//
// Keys are staged 64 at a time (two 32-key tiles), double buffered, one barrier
// per stage.  K and V of the next stage are on their way into registers while
// the current one is computed, and go to LDS at its end.  (As direct-to-LDS
// loads they were waited for in the middle of the stage: the compiler takes the
// transposing reads of V as possible readers of a load in flight and puts
// vmcnt(0) before them.  Head size 64, and blocks of fewer than 4 waves, whose
// share of a stage their registers would not hold, still load that way.)  K rows are 16-byte-chunk XOR-swizzled by row
// (conflict-free fragment reads); V stays in its natural [key][dim] layout and
// the V^T fragments of O^T = V^T P^T come from it by transposing LDS reads
// (lds_read_tr16).  Scores are formed transposed, S^T = K Q^T, with the 32 key
// rows of a tile fed in a permuted order (bits 2 and 3 of the row index
// swapped) so that register e of the score tile holds key 16*(e/8) +
// 8*(lane/32) + e%8 of query lane%32: exactly the operand layout of P^T.  Every
// lane therefore owns one query: the online softmax (running max and sum) lives
// in registers; the max moves only when a score passes it by more than 8
// (log2 units), so the weights stay below 2^8.  P is fed to the MFMA as a
// bf16 pair hi + lo (P - hi), which keeps P V at near-fp32 accuracy.  The
// causal mask is computed from indices, only on tiles that straddle the
// diagonal; tiles past it are never visited (the role the paper's small
// reusable mask plays, Sec. 4.6.1).
//
// A query tile whose keys fit one chunk writes its output directly.
// Otherwise every chunk writes its partial state (running max, sum and
// unnormalised output, in the accumulator layout: coalesced) and a second
// kernel merges the chunks of each query tile in chunk order with the
// log-sum-exp rule, so results do not depend on timing.
//
// Decode: one query per sequence.  Split-KV: a block walks a share of one kv
// head's cache for all the query heads of its group (attn_decode_kernel); the
// last block of a head group to finish merges the shares with the log-sum-exp
// rule.
#include "common.h"
#include "launch.h"

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int key_perm(int r) {  // swap bits 2 and 3
    return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1);
}

constexpr int PF_MAXHB = 8;                  // query heads per block
constexpr int PF_KST = 64;                   // keys per LDS stage

// Query tile and key chunk of work item `item` (longest first): query tile
// qt has nkeys(qt) = L + min(T, 32 (qt + 1)) keys, cut into chunks of
// chunk_keys.  `first` is the item of the tile's chunk 0.
__device__ __forceinline__ void prefill_item(const AttnPrefillArgs& a, int item, int& qt, int& chunk, int& nch,
                                             int& first) {
    const int nqt = (a.T + 31) / 32;
    int base = 0;
    for (qt = nqt - 1; qt > 0; qt--) {
        const int nk = a.L + min(a.T, 32 * (qt + 1));
        const int n = (nk + a.chunk_keys - 1) / a.chunk_keys;
        if (item < base + n) break;
        base += n;
    }
    const int nk = a.L + min(a.T, 32 * (qt + 1));
    nch = (nk + a.chunk_keys - 1) / a.chunk_keys;
    chunk = item - base;
    first = base;
}

template <int D>
__device__ __forceinline__ size_t part_index(const AttnPrefillArgs& a, int row, int item, int wave, int lane) {
    constexpr int NREG = 2 + 16 * (D / 32);
    return ((size_t)(row * a.items + item) * PF_MAXHB + wave) * NREG * 64 + lane;
}

// ML: 1 KB stage loads per wave (K and V together) at most; 0: direct-to-LDS
// loads (blocks of few waves; d = 64, whose smaller registers let two blocks of
// 7 waves share a CU: 700 tokens of Qwen-0.5B 21 us either way, 1500 over 500
// 36 against 40).  Bound by the latency of a stage's chain (scores, softmax, P V) with
// two waves per SIMD: 1.7 us a stage with one block per CU, 2.4 with two
// (d = 128).
template <int D, int ML>
__global__ void __launch_bounds__(64 * PF_MAXHB) attn_prefill_kernel(AttnPrefillArgs a) {
    constexpr int NCH = D / 8;               // 16-byte chunks per K / V row
    constexpr int STB = PF_KST * D * 2;      // bytes of one K or V stage
    constexpr int NT = 2;                    // 32-key tiles per stage
    constexpr int KROWS = 1024 / (2 * D);    // rows per load
    constexpr int NLOAD = PF_KST / KROWS;    // loads per K or V stage
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* const Ks = smem;              // [2][64 keys][D], chunks swizzled
    unsigned char* const Vs = smem + 2 * STB;    // [2][64 keys][D]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HB = blockDim.x / 64;
    const int h = lane >> 5, c = lane & 31;
    const int r = a.nq / a.nkv;
    const int g = blockIdx.y / a.ngrp, hg = blockIdx.y % a.ngrp;
    const int hidx = hg * HB + wave;
    const bool active = hidx < r;
    const int head = g * r + (active ? hidx : 0);
    int qt, chunk, nch, first;
    prefill_item(a, blockIdx.x, qt, chunk, nch, first);
    const int q0 = qt * 32;
    const int nkeys = a.L + min(a.T, q0 + 32);
    const int k0 = chunk * a.chunk_keys, k1 = min(nkeys, k0 + a.chunk_keys);
    const int nst = (k1 - k0 + PF_KST - 1) / PF_KST;
    const uint16_t* kc = a.k_cache + (size_t)g * a.cache_stride_h;
    const uint16_t* vc = a.v_cache + (size_t)g * a.cache_stride_h;

    // ---- stage of 64 keys: 2 NLOAD loads of 1 KB (K, then V), wave w takes
    // loads w, w + HB, ..; load i fills rows KROWS i .. + KROWS - 1; lane l holds
    // chunk l % NCH of its row (for K logical chunk (l % NCH) ^ (row % NCH))
    u32x4 sr[ML ? ML : 1];
    auto stage_src = [&](int i, int st) __attribute__((always_inline)) {
        const bool isv = i >= NLOAD;
        const int row = (isv ? i - NLOAD : i) * KROWS + lane / NCH;
        int slot = k0 + st * PF_KST + row;
        slot = slot < k1 ? slot : k1 - 1;
        const int pc = lane % NCH, lc = isv ? pc : pc ^ (row % NCH);
        return (isv ? vc : kc) + (size_t)slot * D + lc * 8;
    };
    auto stage_dst = [&](int i, int buf) __attribute__((always_inline)) {
        return i >= NLOAD ? Vs + buf * STB + (i - NLOAD) * 1024 : Ks + buf * STB + i * 1024;
    };
    auto load_stage = [&](int st, int buf) __attribute__((always_inline)) {
        if constexpr (ML == 0) {
            for (int i = wave; i < 2 * NLOAD; i += HB)
                __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(stage_src(i, st)),
                                                 (__attribute__((address_space(3))) void*)stage_dst(i, buf), 16, 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < ML; j++) {
                const int i = wave + j * HB;
                if (i < 2 * NLOAD) sr[j] = *reinterpret_cast<const u32x4*>(stage_src(i, st));
            }
        }
    };
    auto store_stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < ML; j++) {
            const int i = wave + j * HB;
            if (i < 2 * NLOAD) *reinterpret_cast<u32x4*>(stage_dst(i, buf) + lane * 16) = sr[j];
        }
    };

    // Q^T fragments (B operand): query q0 + c, dims 16s + 8h .. +8
    bf16x8 qf[D / 16];
    const int qrow = q0 + c;
    const int qload = qrow < a.T ? qrow : a.T - 1;
    load_stage(0, 0);
#pragma unroll
    for (int s = 0; s < D / 16; s++)
        qf[s] = *reinterpret_cast<const bf16x8*>(a.q + ((size_t)qload * a.nq + head) * D + s * 16 + h * 8);

    f32x16 o[D / 32];
#pragma unroll
    for (int i = 0; i < D / 32; i++) o[i] = f32x16{};
    float m = -INFINITY, l = 0.f;
    const int qslot = a.L + qrow;
    const int krow = key_perm(c);
    store_stage(0);
    __syncthreads();
    for (int st = 0; st < nst; st++) {
        const int buf = st & 1;
        if (st + 1 < nst) load_stage(st + 1, buf ^ 1);
        if (active) {
            const unsigned char* K = Ks + buf * STB;
            const __bf16* V = reinterpret_cast<const __bf16*>(Vs + buf * STB);
            // S^T of the wave's 32-key tiles, independent MFMA chains
            f32x16 sc[NT];
#pragma unroll
            for (int t = 0; t < NT; t++) sc[t] = f32x16{};
#pragma unroll
            for (int s = 0; s < D / 16; s++) {
                const int lc = (2 * s + h) ^ (krow % NCH);
#pragma unroll
                for (int t = 0; t < NT; t++) {
                    const bf16x8 kf = *reinterpret_cast<const bf16x8*>(K + (32 * t + krow) * (2 * D) + lc * 16);
                    sc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], sc[t], 0, 0, 0);
                }
            }
            const int kbase = k0 + st * PF_KST;
            const bool diag = kbase + 32 * NT - 1 > a.L + q0;
            float p[16 * NT];
#pragma unroll
            for (int e = 0; e < 16 * NT; e++) p[e] = sc[e / 16][e % 16];
            if (diag) {            // (only the stages that straddle the diagonal)
#pragma unroll
                for (int e = 0; e < 16 * NT; e++) {
                    const int kslot = kbase + 32 * (e / 16) + 16 * ((e % 16) / 8) + 8 * h + (e % 8);
                    if (kslot > qslot) p[e] = -INFINITY;
                }
            }
            float mt = -INFINITY;
#pragma unroll
            for (int e = 0; e < 16 * NT; e++) mt = fmaxf(mt, p[e]);
            mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
            const float m_new = fmaxf(m, mt * a.scale_log2);       // (log2 units)
            // The running max m moves (and o, l are rescaled) only when some
            // lane's scores pass it by more than 8 (log2 units); until then the
            // weights are taken against the older m and stay below 2^8, which
            // the hi + lo split of P carries as well as weights below 1.  While
            // every key so far is masked, m is -inf and the weights are 0.
            if (__builtin_amdgcn_ballot_w64(m_new > m + 8.0f) != 0) {
                const float alpha = exp2_hw(m - (m_new == -INFINITY ? 0.f : m_new));
                l *= alpha;
#pragma unroll
                for (int i = 0; i < D / 32; i++)
#pragma unroll
                    for (int e = 0; e < 16; e++) o[i][e] *= alpha;
                m = m_new;
            }
            const float mb = m == -INFINITY ? 0.f : m;
            float ls[4] = {0.f, 0.f, 0.f, 0.f};          // (four chains)
#pragma unroll
            for (int e = 0; e < 16 * NT; e++) {
                p[e] = exp2_hw(__builtin_fmaf(p[e], a.scale_log2, -mb));
                ls[e % 4] += p[e];
            }
            l += (ls[0] + ls[1]) + (ls[2] + ls[3]);
            // O^T += V^T P^T over the key groups of 16 (tile, step)
#pragma unroll
            for (int ks = 0; ks < 2 * NT; ks++) {
                bf16x8 phi, plo;
#pragma unroll
                for (int j = 0; j < 8; j += 2) {          // pairs: one packed conversion each
                    const bf16x2 hi = __builtin_convertvector(f32x2{p[8 * ks + j], p[8 * ks + j + 1]}, bf16x2);
                    const bf16x2 lo = __builtin_convertvector(
                        f32x2{p[8 * ks + j] - (float)hi[0], p[8 * ks + j + 1] - (float)hi[1]}, bf16x2);
                    phi[j] = hi[0]; phi[j + 1] = hi[1];
                    plo[j] = lo[0]; plo[j + 1] = lo[1];
                }
                // this lane's 8 keys 16 ks + 8 h .. + 7, dim i * 32 + c, by two
                // transposing reads: lane s of its 16-lane group points at key
                // 16 ks + 8 h + s / 4 (+ 4), dims 16 (c / 16) + 4 (s % 4) .. + 3
                const __bf16* vrow = V + (16 * ks + 8 * h + ((lane & 15) >> 2)) * D + 16 * (c >> 4) + 4 * (lane & 3);
#pragma unroll
                for (int i = 0; i < D / 32; i++) {
                    const i16x4 v0 = lds_read_tr16(vrow + i * 32), v1 = lds_read_tr16(vrow + 4 * D + i * 32);
                    const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                    o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, phi, o[i], 0, 0, 0);
                    o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, plo, o[i], 0, 0, 0);
                }
            }
        }
        if (st + 1 < nst) store_stage(buf ^ 1);
        __syncthreads();
    }

    if (!active) return;

    if (nch == 1) {
        // output: dim of register e of block i is i * 32 + 8 (e / 4) + 4 h + e % 4
        if (qrow >= a.T) return;
        const float lt = l + __shfl_xor(l, 32, 64);
        const float inv = (lt > 0.f) ? 1.f / lt : 0.f;
        f16* out = a.out + ((size_t)qrow * a.nq + head) * D;
        bool bad = false;
#pragma unroll
        for (int i = 0; i < D / 32; i++)
#pragma unroll
            for (int e = 0; e < 16; e += 4) {
                f16 v[4];
#pragma unroll
                for (int j = 0; j < 4; j++) v[j] = act_f16(o[i][e + j] * inv, bad);
                *reinterpret_cast<uint2*>(out + i * 32 + 2 * e + 4 * h) = *reinterpret_cast<const uint2*>(v);
            }
        flag_range(a.err, bad);
        return;
    }
    // partial state of this chunk: [row][item][head][m, l, O registers][64 lanes]
    float* pp = a.part + part_index<D>(a, blockIdx.y, blockIdx.x, wave, lane);
    pp[0] = m;
    pp[64] = l;
#pragma unroll
    for (int i = 0; i < D / 32; i++)
#pragma unroll
        for (int e = 0; e < 16; e++) pp[(size_t)(2 + i * 16 + e) * 64] = o[i][e];
}

// Merge of the chunk states of the query tiles with more than one chunk:
// block (query tile, block row, 32-dim slice): thread (wave, lane) merges the
// lane's 16 output registers of the slice over the tile's chunks, in order.
// CB chunks are requested together: 4, or 8 for tiles of more than 8 chunks
// (64 tokens over 4000, 16 chunks; short tiles would only read more).
template <int D, int CB>
__global__ void __launch_bounds__(64 * PF_MAXHB) attn_prefill_merge_kernel(AttnPrefillArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int HB = blockDim.x / 64;
    const int h = lane >> 5, c = lane & 31;
    const int qt = blockIdx.x, row = blockIdx.y, i = blockIdx.z;
    const int r = a.nq / a.nkv;
    const int g = row / a.ngrp, hidx = (row % a.ngrp) * HB + wave;
    const int nqt = (a.T + 31) / 32;
    // first item of tile qt (items run from the last tile down)
    int first = 0;
    for (int t = nqt - 1; t > qt; t--) first += (a.L + min(a.T, 32 * (t + 1)) + a.chunk_keys - 1) / a.chunk_keys;
    const int nch = (a.L + min(a.T, 32 * (qt + 1)) + a.chunk_keys - 1) / a.chunk_keys;
    if (nch == 1 || hidx >= r) return;
    // chunks in groups of CB: the states of a group are requested together,
    // then merged into the running maximum M, sum L and output acc
    float M = -INFINITY, L = 0.f, acc[16] = {};
    for (int ch0 = 0; ch0 < nch; ch0 += CB) {
        float mc[CB], lc[CB], v[CB][16];
#pragma unroll
        for (int j = 0; j < CB; j++) {
            const int ch = ch0 + j < nch ? ch0 + j : nch - 1;
            const float* pp = a.part + part_index<D>(a, row, first + ch, wave, lane);
            mc[j] = pp[0];
            lc[j] = pp[64];
#pragma unroll
            for (int e = 0; e < 16; e++) v[j][e] = pp[(size_t)(2 + i * 16 + e) * 64];
        }
        float Mn = M;
#pragma unroll
        for (int j = 0; j < CB; j++)
            if (ch0 + j < nch) Mn = fmaxf(Mn, mc[j]);
        if (Mn == -INFINITY) continue;
        const float sc = (M == -INFINITY) ? 0.f : exp2f(M - Mn);
        L *= sc;
#pragma unroll
        for (int e = 0; e < 16; e++) acc[e] *= sc;
#pragma unroll
        for (int j = 0; j < CB; j++) {
            if (ch0 + j >= nch || mc[j] == -INFINITY) continue;
            const float w = exp2f(mc[j] - Mn);
            L += w * lc[j];
#pragma unroll
            for (int e = 0; e < 16; e++) acc[e] += w * v[j][e];
        }
        M = Mn;
    }
    const int qrow = qt * 32 + c;
    const float lt = L + __shfl_xor(L, 32, 64);
    if (qrow >= a.T) return;
    const float inv = (lt > 0.f) ? 1.f / lt : 0.f;
    f16* out = a.out + ((size_t)qrow * a.nq + g * r + hidx) * D;
    bool bad = false;
#pragma unroll
    for (int e = 0; e < 16; e += 4) {
        f16 v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = act_f16(acc[e + j] * inv, bad);
        *reinterpret_cast<uint2*>(out + i * 32 + 2 * e + 4 * h) = *reinterpret_cast<const uint2*>(v);
    }
    flag_range(a.err, bad);
}

// ---------------------------------------------------------------- decode

constexpr int MAXR = 8;          // query heads per kv head
constexpr int DEC_W = 8;         // waves per block
constexpr int DEC_ST = 32 * DEC_W;   // keys per stage of a block (32 per wave)

// One block: a contiguous share of the keys of one (row, kv head), all r query
// heads of the group.  Bound by the cache read, so everything is arranged to
// keep loads in flight: the eight waves take 32 keys each of every 256-key
// stage on their own (no barrier in the loop), and a wave's K and V of the
// next stage are on their way into registers while the current one is
// computed.  K goes from memory straight into the MFMA's A operand; V passes
// through LDS, where the transposing read forms V^T.  (With both staged in LDS
// by direct-to-LDS loads, one 64-key chunk per block, a block had nothing in
// flight while it computed, and every chunk cost a launch slot, a partial
// state and its share of the merge.)
//
// Scores S^T = K Q^T and O^T = V^T P^T on the 16x16x32 bf16 MFMA: the heads
// are the columns (padded to 16); the key rows are fed in the order that
// leaves the probabilities in the operand layout of P^T; P is a bf16 pair
// hi + lo.  Every wave keeps a running max, sum and output; the waves meet in
// LDS at the end.  Rows past the share's keys read its last row (in the last
// share the new token's, so V stays finite) and get probability 0.  Hidden slots
// (mask -inf) may hold anything, a NaN of memory that was never written among
// it: their scores are set, not added to, and their V rows become zeros.
//
// With more than one share the blocks store their states (device-coherent, as
// the prefill GEMM's split sums) and count their arrival; the last one merges
// the shares in order, so the result does not depend on timing.  One launch
// instead of two: at these sizes a launch costs as much as the merge.  Whole
// decode before / after this kernel and the GEMV's present form: Qwen-7B, 8 rows
// of up to 8192 keys 121.9 / 86.6 us, Llama-8B, 4 rows of up to 1500 with a mask
// 73.7 / 59.9; the attention alone at the former 39 / 27 us (105 MB of cache).
template <int D>
__global__ void __launch_bounds__(64 * DEC_W) attn_decode_kernel(AttnDecodeArgs a) {
    constexpr int NCK = D / 8, KROWS = 1024 / (2 * D), NV = 32 / KROWS, NS = D / 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ float gst[DEC_W][MAXR][2];
    __shared__ unsigned last_flag;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x / a.nkv, g = blockIdx.x % a.nkv;
    const int ctx = a.ctx_lens ? a.ctx_lens[b] : a.ctx_base + b;
    const int ns = (ctx + DEC_ST) / DEC_ST;                     // stages of ctx + 1 keys
    const int n = min(a.nsplit, ns), part = blockIdx.y;
    if (part >= n) return;
    const int start = (int)((long long)part * ns / n) * DEC_ST;
    const int end = min((int)((long long)(part + 1) * ns / n) * DEC_ST, ctx + 1);
    const int r = a.nq / a.nkv;
    const uint16_t* kc = a.k_cache + (size_t)b * a.stride_b + (size_t)g * a.stride_h;
    const uint16_t* vc = a.v_cache + (size_t)b * a.stride_b + (size_t)g * a.stride_h;
    const float LOG2E = 1.4426950408889634f;
    const int n16 = lane & 15, q4 = lane >> 4;
    unsigned char* const Vst = smem + wave * 32 * D * 2;        // this wave's [32 keys][D], chunks swizzled
    auto vswz = [](int k) { return 2 * ((k >> 3) & 3); };

    // A row n16 of score tile t is key 8 (n16 / 4) + 4 t + n16 % 4 of the
    // wave's 32, so register j of lane (n16, q4) is key 8 q4 + 4 t + j, head n16
    u32x4 kr[2][NS], vr[NV];
    float mk[8];                                                // mask of keys 8 q4 .. + 7
    auto load_stage = [&](int k0) __attribute__((always_inline)) {
        if (a.mask) {
#pragma unroll
            for (int e = 0; e < 8; e++) mk[e] = a.mask[(size_t)b * a.max_seq + min(k0 + 8 * q4 + e, end - 1)];
        }
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const int key = k0 + 8 * (n16 >> 2) + 4 * t + (n16 & 3);
            const uint16_t* src = kc + (size_t)min(key, end - 1) * D + 8 * q4;
#pragma unroll
            for (int s = 0; s < NS; s++) kr[t][s] = *reinterpret_cast<const u32x4*>(src + 32 * s);
        }
#pragma unroll
        for (int i = 0; i < NV; i++) {
            const int key = k0 + i * KROWS + lane / NCK;
            vr[i] = *reinterpret_cast<const u32x4*>(vc + (size_t)min(key, end - 1) * D + (lane % NCK) * 8);
        }
    };
    int k0 = start + 32 * wave;
    u32x4 qw[NS];
    const uint16_t* qsrc = a.q + ((size_t)b * a.nq + g * r + (n16 < r ? n16 : 0)) * D + 8 * q4;
#pragma unroll
    for (int s = 0; s < NS; s++) qw[s] = *reinterpret_cast<const u32x4*>(qsrc + 32 * s);
    load_stage(k0);
    bf16x8 qf[NS];
#pragma unroll
    for (int s = 0; s < NS; s++) qf[s] = __builtin_bit_cast(bf16x8, n16 < r ? qw[s] : u32x4{0u, 0u, 0u, 0u});

    f32x4 o[D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; i++) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    for (; k0 < end; k0 += DEC_ST) {
        f32x4 sacc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < NS; s++) {
            sacc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[0][s]), qf[s], sacc[0], 0, 0, 0);
            sacc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[1][s]), qf[s], sacc[1], 0, 0, 0);
        }
        float ml[8];                                            // (log2 units)
        uint32_t hidden = 0;
        if (a.mask) {
#pragma unroll
            for (int e = 0; e < 8; e++) {
                ml[e] = mk[e] * LOG2E;
                hidden |= (uint32_t)(ml[e] == -INFINITY) << e;
            }
            if (__builtin_amdgcn_ballot_w64(hidden != 0) != 0) {
#pragma unroll
                for (int i = 0; i < NV; i++) {
                    const int row = i * KROWS + lane / NCK;     // lane 16 (row / 8) holds its bit
                    if (__shfl(hidden, 16 * (row >> 3), 64) >> (row & 7) & 1) vr[i] = u32x4{0u, 0u, 0u, 0u};
                }
            }
        }
        // V to LDS (its readers below are this wave alone, so no barrier; a
        // wave's LDS operations are served in order)
#pragma unroll
        for (int i = 0; i < NV; i++) {
            const int row = i * KROWS + lane / NCK;
            *reinterpret_cast<u32x4*>(Vst + (size_t)row * D * 2 + (((lane % NCK) ^ vswz(row)) << 4)) = vr[i];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        load_stage(k0 + DEC_ST);          // (past the end: the share's last row, never used)
        float sv[8];
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            float v = sacc[e / 4][e % 4] * a.scale_log2;
            if (a.mask) v = hidden >> e & 1 ? -INFINITY : v + ml[e];
            v = k0 + 8 * q4 + e < end ? v : -INFINITY;
            sv[e] = v;
            mx = fmaxf(mx, v);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m, mx);
        const float mb = m_new == -INFINITY ? 0.f : m_new;     // (every key so far masked: all weights 0)
        const float alpha = exp2_hw(m - mb);
        bf16x8 phi, plo;
        float ls = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const float pv = exp2_hw(sv[e] - mb);
            ls += pv;
            const __bf16 hi = (__bf16)pv;
            phi[e] = hi;
            plo[e] = (__bf16)(pv - (float)hi);
        }
        ls += __shfl_xor(ls, 16, 64);
        ls += __shfl_xor(ls, 32, 64);
        l = l * alpha + ls;
        m = m_new;
        // O^T += V^T P^T per 16-dim block db: lane (n16, q4) holds V of keys
        // 8 q4 .. + 7, dim 16 db + n16 (two transposing reads: lane n16 of its
        // group points at key 8 q4 + n16 / 4 (+ 4), dims 16 db + 4 (n16 % 4) .. + 3,
        // in their swizzled chunk)
        const uint16_t* Vw = reinterpret_cast<const uint16_t*>(Vst + (size_t)(8 * q4 + (n16 >> 2)) * D * 2);
#pragma unroll
        for (int db = 0; db < D / 16; db++) {
            const int off = (((2 * db + ((n16 & 3) >> 1)) ^ (2 * q4)) << 3) | (4 * (n16 & 1));
            const i16x4 v0 = lds_read_tr16(Vw + off), v1 = lds_read_tr16(Vw + 4 * D + off);
            const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int e = 0; e < 4; e++) o[db][e] *= alpha;
            o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, phi, o[db], 0, 0, 0);
            o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, plo, o[db], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }

    // ---- the waves' states meet in LDS: outputs over the V stages
    __syncthreads();
    float* const ored = reinterpret_cast<float*>(smem);          // [DEC_W][MAXR][D]
    if (n16 < r) {
#pragma unroll
        for (int db = 0; db < D / 16; db++)
            *reinterpret_cast<f32x4*>(ored + (wave * MAXR + n16) * D + 16 * db + 4 * q4) = o[db];
        if (q4 == 0) {
            gst[wave][n16][0] = m;
            gst[wave][n16][1] = l;
        }
    }
    __syncthreads();
    // share state: [row, kv head][share][r heads][D] outputs, then [..][r][2] (max, sum)
    const size_t tile = (size_t)blockIdx.x * a.nsplit;
    unsigned long long* const po = reinterpret_cast<unsigned long long*>(a.part) + tile * r * (D / 2);
    unsigned long long* const pst = reinterpret_cast<unsigned long long*>(a.part) +
                                    (size_t)gridDim.x * a.nsplit * r * (D / 2) + tile * r;
    auto pack = [](float x, float y) { return (unsigned long long)__float_as_uint(y) << 32 | __float_as_uint(x); };
    f16* const out = a.out + ((size_t)b * a.nq + g * r) * D;
    bool bad = false;
    auto put = [&](int idx, float x, float y, float lt) __attribute__((always_inline)) {     // output pair idx
        const f16 h0 = act_f16(lt > 0.f ? x / lt : 0.f, bad), h1 = act_f16(lt > 0.f ? y / lt : 0.f, bad);
        reinterpret_cast<uint32_t*>(out)[idx] =
            (uint32_t)__builtin_bit_cast(uint16_t, h0) | (uint32_t)__builtin_bit_cast(uint16_t, h1) << 16;
    };
    for (int idx = tid; idx < r * (D / 2); idx += 64 * DEC_W) {
        const int i = idx / (D / 2);
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < DEC_W; w++) M = fmaxf(M, gst[w][i][0]);
        float x = 0.f, y = 0.f, lt = 0.f;
#pragma unroll
        for (int w = 0; w < DEC_W; w++) {
            const float sc = gst[w][i][0] == -INFINITY ? 0.f : exp2f(gst[w][i][0] - M);
            const float2 v = *reinterpret_cast<const float2*>(ored + w * MAXR * D + 2 * idx);
            x += sc * v.x;
            y += sc * v.y;
            lt += sc * gst[w][i][1];
        }
        if (n == 1) {
            put(idx, x, y, lt);
        } else {
            __hip_atomic_store(po + (size_t)part * r * (D / 2) + idx, pack(x, y), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (idx % (D / 2) == 0)
                __hip_atomic_store(pst + part * r + i, pack(M, lt), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (n > 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores are complete
        __syncthreads();
        if (tid == 0)
            last_flag = __hip_atomic_fetch_add(a.cnt + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
                        (unsigned)n;
        __syncthreads();
        if (!last_flag) return;
        // the statistics of all shares and the outputs of the first CB are
        // requested together: one memory round trip
        constexpr int CB = 16;
        unsigned long long v[CB];
        auto load_v = [&](int idx, int c0) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < CB; c++)
                v[c] = __hip_atomic_load(po + (size_t)(c0 + c < n ? c0 + c : n - 1) * r * (D / 2) + idx,
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        const int idx0 = tid < r * (D / 2) ? tid : 0;
        unsigned long long s0 = 0;
        if (tid < n * r) s0 = __hip_atomic_load(pst + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        load_v(idx0, 0);
        float2* const st = reinterpret_cast<float2*>(smem);     // [share][r] (max, sum)
        if (tid < n * r) st[tid] = float2{__uint_as_float((unsigned)s0), __uint_as_float((unsigned)(s0 >> 32))};
        for (int i = tid + 64 * DEC_W; i < n * r; i += 64 * DEC_W) {
            const unsigned long long u = __hip_atomic_load(pst + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            st[i] = float2{__uint_as_float((unsigned)u), __uint_as_float((unsigned)(u >> 32))};
        }
        __syncthreads();
        for (int idx = tid; idx < r * (D / 2); idx += 64 * DEC_W) {
            const int i = idx / (D / 2);
            float M = -INFINITY;
            for (int c = 0; c < n; c++) M = fmaxf(M, st[c * r + i].x);
            float x = 0.f, y = 0.f, lt = 0.f;
            for (int c0 = 0; c0 < n; c0 += CB) {
                if (c0 > 0 || idx != tid) load_v(idx, c0);
#pragma unroll
                for (int c = 0; c < CB; c++) {
                    if (c0 + c >= n) break;
                    const float2 s = st[(c0 + c) * r + i];
                    if (s.x == -INFINITY) continue;
                    const float w = exp2f(s.x - M);
                    lt += w * s.y;
                    x += w * __uint_as_float((unsigned)v[c]);
                    y += w * __uint_as_float((unsigned)(v[c] >> 32));
                }
            }
            put(idx, x, y, lt);
        }
    }
    flag_range(a.err, bad);
}

}  // namespace

AttnPrefillPlan attn_prefill_plan(int T, int L, int nq, int nkv, int d, int num_cus) {
    AttnPrefillPlan p;
    const int r = nq / nkv;
    const int hb = r < PF_MAXHB ? r : PF_MAXHB;
    p.ngrp = (r + hb - 1) / hb;
    p.threads = 64 * hb;
    const int nqt = (T + 31) / 32;
    const long long rows = (long long)nkv * p.ngrp;
    const int nreg = 2 + 16 * (d / 32);
    // Key chunk (in stages, at least 2): the one with the least estimated time,
    // in us.  A stage takes a block t, or t2 where blocks share CUs (up to two of
    // 4 waves do) or take turns; a block's start and end count as one stage more;
    // chunks cost the merge launch, its passes over a tile's chunks, and the
    // write and read of their states at about 5.5 TB/s.  Fitted to the chunks of 2 to 32 stages at 16 (T, L) of the
    // Llama-8B, Qwen-7B and Qwen-0.5B layers; against grids of about two blocks
    // per CU, attention and merge: Llama-8B, 1000 tokens 44.1 -> 39.0 us, 64
    // over 4000 33.5 -> 26.1, Qwen-7B, 2011 tokens 114.7 -> 89.2, 100 over 3000
    // 41.1 -> 30.6.
    const double t = d == 64 ? 1.5 : hb > 4 ? 2.2 : 1.7, t2 = (d == 64 ? 1.2 : 1.4) * t;
    const long long slots = (long long)num_cus * (p.threads <= 256 || d == 64 ? 2 : 1);
    const int smax = (L + T + PF_KST - 1) / PF_KST;
    double best = -1.0;
    int cs = 2;
    for (int c = 2;; c += c < 8 ? 1 : c / 4) {
        long long blocks = 0, parts = 0, total = 0;
        for (int qt = 0; qt < nqt; qt++) {
            const int st = (L + std::min(T, 32 * (qt + 1)) + PF_KST - 1) / PF_KST, n = (st + c - 1) / c;
            blocks += n;
            parts += n > 1 ? n : 0;
            total += st;
        }
        blocks *= rows;
        parts *= rows;
        total *= rows;
        const double longest = std::min(c, smax) + 1.0;
        double us = blocks <= num_cus ? t * longest
                    : blocks <= slots ? t2 * longest
                                      : t2 * std::max(longest, (double)(total + blocks) / (double)slots + longest);
        if (parts) us += 3.5 + 0.2 * ((smax + c - 1) / c) + (double)parts * hb * nreg * 512.0 / 5.5e6;
        if (best < 0 || us < best) {
            best = us;
            cs = c;
        }
        if (c >= smax) break;
    }
    p.chunk_keys = PF_KST * cs;
    p.items = 0;
    bool multi = false;
    for (int qt = 0; qt < nqt; qt++) {
        const int n = (L + std::min(T, 32 * (qt + 1)) + p.chunk_keys - 1) / p.chunk_keys;
        p.items += n;
        multi |= n > 1;
    }
    p.merge = multi;
    const size_t per_item = (size_t)rows * PF_MAXHB * nreg * 64 * sizeof(float);
    p.part_bytes = multi ? (size_t)p.items * per_item : 0;
    // chunks are at least 128 keys: a bound that grows with L, for workspace sizing
    p.part_bound = (size_t)nqt * ((L + T + 127) / 128) * per_item;
    p.lds_bytes = (size_t)4 * PF_KST * d * 2;
    return p;
}

template <int D, int ML>
static int launch_prefill(const AttnPrefillArgs& a, const AttnPrefillPlan& p, dim3 grid, hipStream_t stream) {
    // (every wave's share of a stage's loads fits its registers)
    if (ML && p.threads / 64 * ML < 2 * PF_KST * D * 2 / 1024) return -1;
    static LdsLimit lim;
    if (ensure_lds_limit(lim, (const void*)attn_prefill_kernel<D, ML>, p.lds_bytes)) return -1;
    hipLaunchKernelGGL((attn_prefill_kernel<D, ML>), grid, dim3(p.threads), p.lds_bytes, stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_attn_prefill(const AttnPrefillArgs& a, const AttnPrefillPlan& p, hipStream_t stream) {
    if (p.items < 1 || (p.part_bytes && !a.part)) return -1;
    AttnPrefillArgs b = a;
    b.chunk_keys = p.chunk_keys;
    b.ngrp = p.ngrp;
    b.items = p.items;
    const dim3 grid(p.items, a.nkv * p.ngrp);
    const dim3 mgrid((a.T + 31) / 32, a.nkv * p.ngrp, a.d / 32);
    if (a.d != 128 && a.d != 64) return -1;
    int rc;
    if (a.d == 64) rc = launch_prefill<64, 0>(b, p, grid, stream);
    else rc = p.threads >= 256 ? launch_prefill<128, 8>(b, p, grid, stream) : launch_prefill<128, 0>(b, p, grid, stream);
    if (rc) return rc;
    if (p.merge) {
        const bool many = a.L + a.T > 8 * p.chunk_keys;
        auto fn = a.d == 128 ? (many ? attn_prefill_merge_kernel<128, 8> : attn_prefill_merge_kernel<128, 4>)
                             : (many ? attn_prefill_merge_kernel<64, 8> : attn_prefill_merge_kernel<64, 4>);
        hipLaunchKernelGGL(fn, mgrid, dim3(p.threads), 0, stream, b);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Shares per (row, kv head): the count with the least estimated time.  A stage
// costs a block about 1.3 us (a memory round trip and its arithmetic), a
// second share the hand-off (store, count, read back: three round trips) and a
// little for every state merged.
int attn_decode_splits(int B, int nkv, int max_ctx, int num_cus) {
    const int stages = (int)(((long long)max_ctx + DEC_ST) / DEC_ST);
    int best = 1;
    double best_cost = -1.0;
    for (int n = 1; n <= stages && (n == 1 || (long long)B * nkv * n <= num_cus); n++) {
        const long long rounds = ((long long)B * nkv * n + num_cus - 1) / num_cus;
        const double cost = 1.3 * rounds * ((stages + n - 1) / n) + (n > 1 ? 3.0 + 0.08 * n : 0.0);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = n;
        }
    }
    return best;
}

int launch_attn_decode(const AttnDecodeArgs& a, hipStream_t stream) {
    const int r = a.nq / a.nkv;
    if (r > MAXR || a.nsplit < 1 || (a.nsplit > 1 && (!a.part || !a.cnt))) return -1;
    const dim3 grid(a.B * a.nkv, a.nsplit);
    // V stages of the waves; over them their outputs, then the shares' statistics
    const size_t lds = std::max({(size_t)DEC_W * 32 * a.d * 2, (size_t)DEC_W * MAXR * a.d * 4, (size_t)a.nsplit * r * 8});
    static LdsLimit lim128, lim64;
    if (a.d == 128) {
        if (ensure_lds_limit(lim128, (const void*)attn_decode_kernel<128>, lds)) return -1;
        hipLaunchKernelGGL(attn_decode_kernel<128>, grid, dim3(64 * DEC_W), lds, stream, a);
    } else if (a.d == 64) {
        if (ensure_lds_limit(lim64, (const void*)attn_decode_kernel<64>, lds)) return -1;
        hipLaunchKernelGGL(attn_decode_kernel<64>, grid, dim3(64 * DEC_W), lds, stream, a);
    } else {
        return -1;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int load_attention() { return load_code((const void*)attn_decode_kernel<128>); }
