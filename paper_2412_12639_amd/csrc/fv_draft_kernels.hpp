// Kernels of the drafting phase (the SAR head of the paper: sections "Framework and Computational
// Process", "Coupled Sequential Glancing Distillation", "Custom-Designed Decoding Tree"; Appendix
// "Tree Structure") that the verification step does not already have: input assembly, the LSTM
// cell, the relaxed causal mask, top-m selection and the expansion of the static tree.  The weight
// multiplications, the attention and the decoder-block epilogues are the verification step's kernels.
//
// Rows of a drafting phase are numbered 0..255 ("phase rows"): first the chain of pairs committed
// since the last phase, then the rows of every tree pass.  A phase row's K/V sits in cache slot
// L0 + row, its 256-bit visibility mask is over phase rows.  "Output rows" are the phase rows plus
// FV_DRAFT_KMAX history slots (ids 256..) that keep the predicted feature and top list of the last
// committed rows of earlier phases.
#pragma once
#include "fv_device.hpp"
#include "fv_types.hpp"
#include <float.h>

// ---- per-phase tables (device copies of what the host planned from the static tree)
struct DraftTables {
    const int32_t* feat_src;   // [256] phase row -> output row id whose predicted feature it takes in, or -1 - e: row e of the external features
    const int32_t* tok_node;   // [256] phase row -> tree node whose token it takes in, or -1: tok_val
    const int32_t* tok_val;    // [256] token given by the host (committed pairs)
    const int32_t* pred;       // [256] phase row before this one on its path (-1: none; the committed prefix is visible anyway)
    const int32_t* lpred;      // [256] row whose LSTM state it continues (FV_DRAFT_STATE_COMMITTED: the last committed row)
    const int32_t* block;      // [256] block id
    const int32_t* pos;        // [256] rotary position
    const int32_t* lvl_rows;   // [256] rows of each pass grouped by LSTM level (pass-local indices)
    const int32_t* node_gen;   // [256] tree node -> output row id whose top list holds its token
    const int32_t* node_rank;  // [256] tree node -> rank in that list
    const int32_t* exp_list;   // [256] tree nodes whose token comes from a list (all but the root)
};

// ============================================================================ mask, positions, rotary table
// Relaxed causal mask (section "Custom-Designed Decoding Tree"): a row sees its predecessors on its
// path and every row of its own block; the rows of a block are always rows of one pass.
struct DraftIngestArgs {
    DraftTables tab;
    int r0, n, Tp, half_d;
    int chain;               // the rows follow each other from row 0 on: no walk
    double log2_base;
    uint64_t* mask;          // [Tp][4]
    float2* rope_cs;         // [Tp][half_d]
};

__device__ __forceinline__ void draft_ingest_rows(const DraftIngestArgs& a, int blk) {   // four rows
    const int tid = threadIdx.x;
    const int t0 = blk * 4, t1 = (t0 + 4 < a.Tp) ? t0 + 4 : a.Tp;
    for (int t = t0 + tid; t < t1; t += 256) {
        uint64_t m[4] = {0, 0, 0, 0};
        if (t < a.n && a.chain) {
            for (int w = 0; w < 4; ++w) { const int k = t + 1 - 64 * w; m[w] = k <= 0 ? 0ull : k >= 64 ? ~0ull : (1ull << k) - 1ull; }
        } else if (t < a.n) {
            const int r = a.r0 + t;
            int j = r, guard = 0;
            while (j >= 0 && j < FV_MAX_TREE && guard++ < FV_MAX_TREE) {   // the host made pred[j] < j; the guard bounds the walk anyway
                m[j >> 6] |= 1ull << (j & 63);
                j = a.tab.pred[j];
            }
            const int b = a.tab.block[r];
            for (int q = a.r0; q < a.r0 + a.n; ++q)
                if (a.tab.block[q] == b) m[q >> 6] |= 1ull << (q & 63);
        }
        for (int w = 0; w < 4; ++w) a.mask[t * 4 + w] = m[w];
    }
    const int n = t1 * a.half_d;
    for (int e = t0 * a.half_d + tid; e < n; e += 256) {
        const int t = e / a.half_d, i = e % a.half_d;
        const int p = (t < a.n) ? a.tab.pos[a.r0 + t] : 0;
        const double inv_freq = exp2(-(double)i / (double)a.half_d * a.log2_base);
        double s, c;
        sincos((double)p * inv_freq, &s, &c);
        a.rope_cs[e] = make_float2((float)c, (float)s);
    }
}

// ============================================================================ input rows
// z = [feature ; embedding of the token one step ahead]  (width 2h), as the vector-major input of
// the first LSTM layer's input multiplication.  Pad columns are zero.
struct DraftInArgs {
    DraftTables tab;
    const float* fout;        // [256 + KMAX][h] predicted features by output row id
    const float* ext;         // external features [..][h] (true features of committed pairs), may be null
    const int32_t* top_tok;   // [256 + KMAX][FV_DRAFT_MMAX] top lists by output row id: a node's token is entry node_rank of row node_gen's
    const void* table;        // embedding [V][h]
    void* xz;                 // [2h/E][Tp][E]
    uint32_t* chain; int chain_words;   // exchange area of the chain launches to clear (0 words: none)
    int r0, n, Tp, h, vocab;
};

// previous hidden state of every row of a level -> vector-major input of the recurrent multiplication
struct LstmGatherArgs {
    DraftTables tab;
    const float* state;   // this layer's state rows
    void* xprev;          // [h/E][Tpl][E]
    int r0, l0, n_lvl, Tpl, h;
};
template <typename EL>
__device__ __forceinline__ void lstm_gather(const LstmGatherArgs& a, size_t idx) {
    const int i = (int)(idx % a.Tpl);
    const int f0 = (int)(idx / a.Tpl) * 4;
    if (f0 >= a.h) return;
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < a.n_lvl) {
        const int r = a.r0 + a.tab.lvl_rows[a.l0 + i];
        x = *(const float4*)(a.state + ((size_t)a.tab.lpred[r] * 2) * a.h + f0);
    }
    store4_act<EL>(a.xprev, a.Tpl, f0, i, x.x, x.y, x.z, x.w);
}

// What a tree pass whose levels go in one launch a layer needs besides, of both layers (the first level's predecessors are rows of earlier passes): their
// states, and the statistics that the launch of layer 1 adds to, cleared.
struct DraftLevelArgs { LstmGatherArgs layer[2]; float* ssq; int n_ssq, n_gather; };   // n_gather workgroups a layer; 0: none

// The start of a pass, input rows, ingest and first predecessors side by side in one launch (they do not depend on each other; a small launch is 5 us
// with its gap): the first n_in workgroups take 256 four-feature groups each, the next Tp / 4 four rows' masks and rotary entries, then come the
// predecessors' states, the others clear padding.
template <typename EL>
static __global__ __launch_bounds__(256) void k_draft_begin(DraftInArgs a, DraftIngestArgs ia, int n_in, DraftLevelArgs lv, PadArgs pa) {
    if ((int)blockIdx.x >= n_in + ia.Tp / 4) {
        int b = blockIdx.x - n_in - ia.Tp / 4;
        if (b >= 2 * lv.n_gather) { clear_pads(pa, (b - 2 * lv.n_gather) * 256 + threadIdx.x); return; }
        for (int i = b * 256 + threadIdx.x; i < lv.n_ssq; i += 2 * lv.n_gather * 256) lv.ssq[i] = 0.f;
        const int l = b >= lv.n_gather;
        lstm_gather<EL>(lv.layer[l], (size_t)(b - l * lv.n_gather) * 256 + threadIdx.x);
        return;
    }
    if ((int)blockIdx.x >= n_in) { draft_ingest_rows(ia, blockIdx.x - n_in); return; }
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    for (size_t i = idx; i < (size_t)a.chain_words; i += (size_t)n_in * 256) a.chain[i] = 0u;
    const int t = (int)(idx % a.Tp);
    const int f0 = (int)(idx / a.Tp) * 4;
    if (f0 >= 2 * a.h) return;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (t < a.n) {
        const int r = a.r0 + t;
        if (f0 < a.h) {
            const int src = a.tab.feat_src[r];
            const float* p = (src >= 0) ? a.fout + (size_t)src * a.h : a.ext + (size_t)(-1 - src) * a.h;
            const float4 x = *(const float4*)(p + f0);
            v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        } else {
            const int nd = a.tab.tok_node[r];
            int tok = (nd >= 0) ? a.top_tok[(size_t)a.tab.node_gen[nd] * FV_DRAFT_MMAX + a.tab.node_rank[nd]] : a.tab.tok_val[r];
            if (tok < 0 || tok >= a.vocab) tok = 0;   // only after a non-finite row, which fails the phase anyway
            const size_t base = (size_t)tok * a.h + (f0 - a.h);
            if constexpr (Tr<EL>::E == 8) {
                const uint2 u = *(const uint2*)((const uint16_t*)a.table + base);
                const uint4 w = make_uint4(u.x, u.y, 0u, 0u);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = Tr<EL>::at(w, c);
            } else {
                const uint4 w = *(const uint4*)((const float*)a.table + base);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = Tr<EL>::at(w, c);
            }
        }
    }
    store4_act<EL>(a.xz, a.Tp, f0, t, v[0], v[1], v[2], v[3]);
}

// ============================================================================ LSTM
// State rows: [257][2][h] fp32 per layer (h then c); row 256 is the state after the last committed pair.
// One level = the rows of a pass whose predecessors' states are all known; level rows are listed in
// lvl_rows[l0 .. l0 + n_lvl).

template <typename EL>
static __global__ __launch_bounds__(256) void k_lstm_gather(LstmGatherArgs a) { lstm_gather<EL>(a, (size_t)blockIdx.x * 256 + threadIdx.x); }

// gates = G_in[row] + G_rec[level row] + bias (rows ordered input, forget, cell, output);
// c' = sigmoid(f) c + sigmoid(i) tanh(g);  h' = sigmoid(o) tanh(c').
// LAYER 0: h' also becomes the row's column of the second layer's input.
// LAYER 1: h' is the decoder block's residual stream x; also x * gain (the un-normalised input of the
// q/k/v multiplication) and the per-strip sums of squares of x.
struct LstmCellArgs {
    DraftTables tab;
    const float* g_in;    // [Tp][4h]
    const float* g_rec;   // [Tpl][4h]
    const float* bias;    // [4h]
    float* state;         // this layer's state rows
    void* xnext;          // LAYER 0: [h/E][Tp][E]
    float* x;             // LAYER 1: [h/4][Tp][4]
    void* xb;             // LAYER 1: [h/E][Tp][E]
    const float* gain;    // LAYER 1: [h]
    float* ssq;           // LAYER 1: [h/32][Tp]
    int r0, l0, n_lvl, Tp, h;
};

__device__ __forceinline__ float fv_sigmoid(float x) { return 1.f / (1.f + expf(-x)); }

template <typename EL, int LAYER>
static __global__ __launch_bounds__(256) void k_lstm_cell(LstmCellArgs a) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int q = a.h / 4;                 // 4-feature groups per row; 8 consecutive lanes share a 32-feature strip
    const int i = (int)(idx / q);
    const int f0 = (int)(idx % q) * 4;
    if (i >= a.n_lvl) return;              // whole strips leave together: h is a multiple of 64
    const int t = a.tab.lvl_rows[a.l0 + i];
    const int r = a.r0 + t;
    const size_t H = a.h;
    const float* gi = a.g_in + (size_t)t * 4 * H;
    const float* gr = a.g_rec + (size_t)i * 4 * H;
    float4 g[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float4 u = *(const float4*)(gi + k * H + f0), w = *(const float4*)(gr + k * H + f0), b = *(const float4*)(a.bias + k * H + f0);
        g[k] = make_float4(u.x + w.x + b.x, u.y + w.y + b.y, u.z + w.z + b.z, u.w + w.w + b.w);
    }
    const float4 cp = *(const float4*)(a.state + ((size_t)a.tab.lpred[r] * 2 + 1) * H + f0);
    const float gin[4] = {g[0].x, g[0].y, g[0].z, g[0].w}, gf[4] = {g[1].x, g[1].y, g[1].z, g[1].w};
    const float gg[4] = {g[2].x, g[2].y, g[2].z, g[2].w}, go[4] = {g[3].x, g[3].y, g[3].z, g[3].w};
    const float cprev[4] = {cp.x, cp.y, cp.z, cp.w};
    float hn[4], cn[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        cn[c] = fv_sigmoid(gf[c]) * cprev[c] + fv_sigmoid(gin[c]) * tanhf(gg[c]);
        hn[c] = fv_sigmoid(go[c]) * tanhf(cn[c]);
    }
    *(float4*)(a.state + ((size_t)r * 2) * H + f0) = make_float4(hn[0], hn[1], hn[2], hn[3]);
    *(float4*)(a.state + ((size_t)r * 2 + 1) * H + f0) = make_float4(cn[0], cn[1], cn[2], cn[3]);
    if constexpr (LAYER == 0) {
        store4_act<EL>(a.xnext, a.Tp, f0, t, hn[0], hn[1], hn[2], hn[3]);
    } else {
        ((float4*)a.x)[(size_t)(f0 >> 2) * a.Tp + t] = make_float4(hn[0], hn[1], hn[2], hn[3]);
        const float4 gn = *(const float4*)(a.gain + f0);
        store4_act<EL>(a.xb, a.Tp, f0, t, hn[0] * gn.x, hn[1] * gn.y, hn[2] * gn.z, hn[3] * gn.w);
        float ssq = hn[0] * hn[0] + hn[1] * hn[1] + hn[2] * hn[2] + hn[3] * hn[3];
        ssq += __shfl_xor(ssq, 1);
        ssq += __shfl_xor(ssq, 2);
        ssq += __shfl_xor(ssq, 4);
        if ((f0 & 31) == 0) a.ssq[(size_t)(f0 >> 5) * a.Tp + t] = ssq;
    }
}

// state after the last committed pair <- state of phase row `row` (both layers are laid out back to back); not if *aborted
// (a chain launch gave up: the rows' states are not there)
// The call's error words go to the host's memory with it.
// (finite_only: not if the pass had values that are no numbers either: the call then runs again in smaller pieces)
struct StateKeepArgs { float* state0; float* state1; const uint32_t* aborted; const int32_t* bad; int32_t* bad_out; int row, h, finite_only; };
static __global__ __launch_bounds__(256) void k_state_keep(StateKeepArgs a) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx < 3) { a.bad_out[idx] = a.bad[idx]; __threadfence_system(); }
    if (idx >= 2 * a.h || *a.aborted || (a.finite_only && a.bad[0])) return;
    a.state0[(size_t)FV_MAX_TREE * 2 * a.h + idx] = a.state0[(size_t)a.row * 2 * a.h + idx];
    a.state1[(size_t)FV_MAX_TREE * 2 * a.h + idx] = a.state1[(size_t)a.row * 2 * a.h + idx];
}

// ============================================================================ outputs of a pass
// predicted feature rows: the block's residual stream after its MLP, fp32 [256 + KMAX][h] by output row id
struct DraftOutArgs { const float* x; float* fout; int r0, n, Tp, h; };
__device__ __forceinline__ void draft_out_row(const DraftOutArgs& a, int t) {
    for (int q = threadIdx.x; q < a.h / 4; q += blockDim.x)   // four features a thread, a whole row of 4096 at once
        ((float4*)(a.fout + (size_t)(a.r0 + t) * a.h))[q] = ((const float4*)a.x)[(size_t)q * a.Tp + t];
}

// Top-m of one row of logits: descending value, lower token id first among equals (a total order, so
// the result is unique).  One workgroup of 1024 threads per row; a thread keeps 32 values in registers
// (vocabulary <= 32768).  The second best of every wavefront's 64 per-thread bests gives 32 values that
// reach the smallest of these sixteen, so that one is a threshold that at least 32 values reach: the
// values that reach it (usually about a hundred) are collected in LDS and ranked by counting.  What bounds it is the chain of these steps in one
// compute unit; with 64-bit keys through LDS in the reductions and three tests a value a row took 14.3 us, now 9.4.  If there
// are more than 256 of them (many equal logits), the list is instead drawn one winner per round.
// A row that holds a NaN or an infinity has no order: its list is filled with -1 and *bad is set.
struct TopmArgs {
    const float* logits;   // [n][Vpad] (row t of this pass)
    int32_t* top_tok;      // [256 + KMAX][FV_DRAFT_MMAX] by output row id
    float* top_val;
    int32_t* bad;          // set to 1 if some row is non-finite
    const int32_t* gate;   // not null: nothing is written if gate[0] or gate[2] is set (a long commit that came to nothing)
    int r0, n, V, Vpad, m;
};

#define FV_TOPM_THREADS 1024
#define FV_TOPM_FAST 256   // candidates the counting path holds

// (value, token id) as one 64-bit integer, larger = earlier in the list; v is finite and not -0.  0 = no value.
__device__ __forceinline__ unsigned long long topm_key(float v, int i) {
    uint32_t u = __float_as_uint(v);
    u ^= (u >> 31) ? 0xFFFFFFFFu : 0x80000000u;
    return ((unsigned long long)u << 32) | (uint32_t)(0x7FFFFFFF - i);
}
__device__ __forceinline__ float topm_key_value(unsigned long long key) {
    uint32_t u = (uint32_t)(key >> 32);
    u ^= (u >> 31) ? 0x80000000u : 0xFFFFFFFFu;
    return __uint_as_float(u);
}
__device__ __forceinline__ int topm_key_token(unsigned long long key) { return 0x7FFFFFFF - (int)(uint32_t)key; }
__device__ __forceinline__ unsigned long long topm_wave_max(unsigned long long k) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const unsigned long long o = ((unsigned long long)(uint32_t)__shfl_xor((int)(k >> 32), off) << 32) | (uint32_t)__shfl_xor((int)(uint32_t)k, off);
        k = o > k ? o : k;
    }
    return k;
}

// (workgroups n .. 2n-1 write the predicted feature rows, which wait for nothing the top lists do)
static __global__ __launch_bounds__(FV_TOPM_THREADS) void k_topm(TopmArgs a, DraftOutArgs oa) {
    if (a.gate && (a.gate[0] || a.gate[2])) return;
    if ((int)blockIdx.x >= a.n) { draft_out_row(oa, blockIdx.x - a.n); return; }
    __shared__ unsigned long long wave_key[16];
    __shared__ float wave_best[16];
    __shared__ unsigned long long cand[FV_TOPM_FAST];
    __shared__ int rank_of[FV_TOPM_FAST];
    __shared__ int n_cand, any_bad;
    const int t = blockIdx.x, tid = threadIdx.x, wave = tid >> 6;
    const float* row = a.logits + (size_t)t * a.Vpad;
    if (tid == 0) { n_cand = 0; any_bad = 0; }
    if (tid < FV_TOPM_FAST) rank_of[tid] = 0;
    float x[32];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int v = (tid + FV_TOPM_THREADS * k) * 4;
        const float4 q = (v < a.V) ? *(const float4*)(row + v) : make_float4(0.f, 0.f, 0.f, 0.f);   // Vpad is a multiple of 32
        x[4 * k] = q.x + 0.f; x[4 * k + 1] = q.y + 0.f; x[4 * k + 2] = q.z + 0.f; x[4 * k + 3] = q.w + 0.f;   // -0 -> +0: equal values, one key
    }
    auto token_of = [&](int e) { return (tid + FV_TOPM_THREADS * (e >> 2)) * 4 + (e & 3); };   // ascending in e
    // One pass: the thread's largest value, and a sum of zeros that a NaN or an infinity anywhere turns into a NaN.  What lies behind the vocabulary is the
    // lowest number: it is no token's, and the list below looks at token ids.
    float bv = -FLT_MAX, zero = 0.f;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        x[e] = token_of(e) < a.V ? x[e] : -FLT_MAX;
        zero = fmaf(x[e], 0.f, zero);
        bv = fmaxf(bv, x[e]);
    }
    const bool bad = !(zero == 0.f);
    // the wavefront's best and second best of its 64 thread bests
    const float w1 = wave_max(bv);
    const unsigned long long at1 = __ballot(bv == w1);
    const float w2 = wave_max((at1 != 0ull && (tid & 63) == __ffsll((long long)at1) - 1) ? -FLT_MAX : bv);
    if ((tid & 63) == 0) wave_best[wave] = w2;
    if (__any(bad) && (tid & 63) == 0) any_bad = 1;   // written before the barrier, read after it (only ever set to 1)
    __syncthreads();
    int32_t* out_t = a.top_tok + (size_t)(a.r0 + t) * FV_DRAFT_MMAX;
    float* out_v = a.top_val + (size_t)(a.r0 + t) * FV_DRAFT_MMAX;
    if (tid < FV_DRAFT_MMAX) { out_t[tid] = -1; out_v[tid] = 0.f; }   // fewer than m tokens, or a non-finite row
    if (any_bad) {
        if (tid == 0) *a.bad = 1;
        return;
    }
    float thr = wave_best[0];
#pragma unroll
    for (int w = 1; w < 16; ++w) thr = fminf(thr, wave_best[w]);   // the lowest number if some wavefront has fewer than two values: everything is a candidate
    if (bv >= thr) {
#pragma unroll
        for (int e = 0; e < 32; ++e)
            if (x[e] >= thr) {
                const int i = token_of(e);
                const int pos = i < a.V ? atomicAdd(&n_cand, 1) : FV_TOPM_FAST;
                if (pos < FV_TOPM_FAST) cand[pos] = topm_key(x[e], i);
            }
    }
    __syncthreads();
    const int C = n_cand;
    if (C <= FV_TOPM_FAST) {
        // rank by counting: 64 candidates at a time, a sixteenth of the comparisons per wavefront
        for (int c0 = 0; c0 < C; c0 += 64) {
            const int c = c0 + (tid & 63);
            if (c < C) {
                const unsigned long long key = cand[c];
                int ahead = 0;
                for (int j = wave; j < C; j += 16) ahead += cand[j] > key ? 1 : 0;
                if (ahead) atomicAdd(&rank_of[c], ahead);
            }
        }
        __syncthreads();
        if (tid < C) {
            const int r = rank_of[tid];
            if (r < a.m && r < FV_DRAFT_MMAX) { out_t[r] = topm_key_token(cand[tid]); out_v[r] = topm_key_value(cand[tid]); }
        }
        return;
    }
    // many values reach the threshold (equal logits): one winner per round, each thread offering its best value
    // that comes after the last winner
    unsigned long long last = ~0ull;
    const int rounds = a.m < FV_DRAFT_MMAX ? a.m : FV_DRAFT_MMAX;
    for (int round = 0; round < rounds; ++round) {
        unsigned long long offer = 0ull;
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const int i = token_of(e);
            const unsigned long long k = i < a.V ? topm_key(x[e], i) : 0ull;
            offer = (k < last && k > offer) ? k : offer;
        }
        const unsigned long long w = topm_wave_max(offer);
        __syncthreads();   // the previous round's wave_key has been read by everyone
        if ((tid & 63) == 0) wave_key[wave] = w;
        __syncthreads();
        unsigned long long win = wave_key[0];
#pragma unroll
        for (int q = 1; q < 16; ++q) win = wave_key[q] > win ? wave_key[q] : win;
        if (win == 0ull) break;   // fewer than m tokens
        if (tid == 0) { out_t[round] = topm_key_token(win); out_v[round] = topm_key_value(win); }
        last = win;
    }
}

// tokens of the tree nodes a pass generates: node_tok[i] = top list of its generating row at its rank
// (and the call's error words), into the host's memory
struct ExpandArgs { DraftTables tab; const int32_t* top_tok; const int32_t* bad; int32_t* node_tok; int32_t* bad_out; int n; };
static __global__ __launch_bounds__(256) void k_draft_expand(ExpandArgs a) {
    const int j = threadIdx.x;   // one workgroup: at most 256 nodes
    if (j < 3) a.bad_out[j] = a.bad[j];
    if (j < a.n) {
        const int i = a.tab.exp_list[j];
        a.node_tok[i] = a.top_tok[(size_t)a.tab.node_gen[i] * FV_DRAFT_MMAX + a.tab.node_rank[i]];
    }
    __threadfence_system();
}

// History of the last k-1 committed rows' outputs (predicted feature, top list), kept across phases in
// output rows 256 .. 256+k-2.  With C = [history, chain rows 0..n_prev-1 of the phase that ends], the new
// history is C[n_prev .. n_prev+k-2].  A new entry j only reads entries above j, so one workgroup moves
// them in ascending order.
struct HistArgs { float* fout; int32_t* top_tok; float* top_val; int n_prev, k, h; };
static __global__ __launch_bounds__(256) void k_draft_hist(HistArgs a) {
    for (int j = 0; j < a.k - 1; ++j) {
        const int c = a.n_prev + j;
        const int src = (c < a.k - 1) ? FV_MAX_TREE + c : c - (a.k - 1);
        const int dst = FV_MAX_TREE + j;
        for (int q0 = threadIdx.x; q0 < a.h / 4; q0 += 4 * 256) {   // four vectors read before the first is stored
            float4 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = ((const float4*)(a.fout + (size_t)src * a.h))[q0 + k * 256 < a.h / 4 ? q0 + k * 256 : q0];
#pragma unroll
            for (int k = 0; k < 4; ++k) if (q0 + k * 256 < a.h / 4) ((float4*)(a.fout + (size_t)dst * a.h))[q0 + k * 256] = v[k];
        }
        if (threadIdx.x < FV_DRAFT_MMAX) {
            a.top_tok[dst * FV_DRAFT_MMAX + threadIdx.x] = a.top_tok[src * FV_DRAFT_MMAX + threadIdx.x];
            a.top_val[dst * FV_DRAFT_MMAX + threadIdx.x] = a.top_val[src * FV_DRAFT_MMAX + threadIdx.x];
        }
        __syncthreads();
    }
}

// The last `keep` rows of a commit's pass become the phase's rows 0 .. keep-1, the k-1 rows in front of them the history: predicted feature, top
// list and logits, and the last row's states.  Rows move by s, which is no less than keep, so only history rows are read where others are written,
// and a workgroup that writes one of those has moved it first.  Grid: keep + k - 1.
struct DraftSliceArgs { float* fout; int32_t* top_tok; float* top_val; float* logits; float* state[2]; const int32_t* bad; int s, keep, k, h, Vpad; };
static __global__ __launch_bounds__(256) void k_draft_slice(DraftSliceArgs a) {
    if (a.bad[0] || a.bad[2]) return;
    const int b = blockIdx.x, tid = threadIdx.x, hist0 = a.s - (a.k - 1);
    const int r = b < a.keep ? b : hist0 + (b - a.keep);   // the row this workgroup writes, or only takes into the history
    if (b >= a.keep && r < a.keep) return;
    const bool hist = r >= hist0 && r < a.s;
    float4* const f = (float4*)a.fout;
    const size_t hq = a.h / 4;
    for (size_t q = tid; q < hq; q += 256) {
        if (hist) f[(size_t)(FV_MAX_TREE + r - hist0) * hq + q] = f[(size_t)r * hq + q];
        if (b < a.keep) f[(size_t)r * hq + q] = f[(size_t)(a.s + r) * hq + q];
    }
    if (tid < FV_DRAFT_MMAX) {
        if (hist) {
            a.top_tok[(FV_MAX_TREE + r - hist0) * FV_DRAFT_MMAX + tid] = a.top_tok[r * FV_DRAFT_MMAX + tid];
            a.top_val[(FV_MAX_TREE + r - hist0) * FV_DRAFT_MMAX + tid] = a.top_val[r * FV_DRAFT_MMAX + tid];
        }
        if (b < a.keep) {
            a.top_tok[r * FV_DRAFT_MMAX + tid] = a.top_tok[(a.s + r) * FV_DRAFT_MMAX + tid];
            a.top_val[r * FV_DRAFT_MMAX + tid] = a.top_val[(a.s + r) * FV_DRAFT_MMAX + tid];
        }
    }
    if (b >= a.keep) return;
    const float4* const from = (const float4*)(a.logits + (size_t)(a.s + r) * a.Vpad);   // Vpad is a multiple of 32
    float4* const to = (float4*)(a.logits + (size_t)r * a.Vpad);
    for (int q = tid; q < a.Vpad / 4; q += 256) to[q] = from[q];
    if (r == a.keep - 1)
        for (int l = 0; l < 2; ++l)
            for (int i = tid; i < 2 * a.h; i += 256) a.state[l][(size_t)r * 2 * a.h + i] = a.state[l][(size_t)(a.s + r) * 2 * a.h + i];
}

// K and V of n slots <- 0: what a pass left there that is run again in pieces.  Its rows may be no numbers, and a piece reads whole blocks of 32 keys, the
// slots behind its own rows masked, which a value that is no number survives.
struct ClearSlotsArgs { void* kcache; void* vcache; int slot0, n, Hkv, S_pad; };
template <typename EL, int D>
static __global__ __launch_bounds__(256) void k_draft_clear_slots(ClearSlotsArgs a) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int f = (int)(idx % D), kh = (int)(idx / D % a.Hkv), j = (int)(idx / D / a.Hkv);
    if (j >= a.n) return;
    const size_t slab = (size_t)kh * a.S_pad * D * Tr<EL>::ESZ;
    st_elem<EL>((char*)a.kcache + slab, kcache_index<EL, D>(a.slot0 + j, f), 0.f);
    st_elem<EL>((char*)a.vcache + slab, vcache_index<EL, D>(a.slot0 + j, f), 0.f);
}

// plain fill (pad columns of activation buffers after a change of the row padding)
static __global__ __launch_bounds__(256) void k_draft_fill(uint32_t* p, uint32_t v, size_t n) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}
