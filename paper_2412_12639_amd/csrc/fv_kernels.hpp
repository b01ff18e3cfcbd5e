// Kernels of one tree-verification step (paper, section "Custom-Designed Decoding Tree":
// the target LLM checks every node of the draft tree in one pass under tree attention,
// then the longest greedily-accepted path is kept).  Layouts are described in
// fv_device.hpp.  Every kernel checks its own bounds; the host checks shapes first.
#pragma once
#include "fv_device.hpp"
#include "fv_types.hpp"
#include <float.h>

// ============================================================================ ingest
// Tree ingest: ancestor sets, positions, rotary table.  One block.
// mask[i] = mask[parent[i]] | bit(i), built by walking the parent chain (at most
// depth steps); position of node i = L + depth[i]  (node i continues the sequence
// prefix ++ root path, so it sits depth[i] places after the root at position L).
struct IngestArgs {
    const int32_t* tok_in;   // [3][cap]: tokens, parent, depth
    int32_t* tok_out;        // tok_in is host memory: the copy that later kernels read, or null
    const double* unif_in;   // non-greedy step, host memory: [2][cap] uniforms, to unif_out; or null
    double* unif_out;
    int cap, T, Tp, L, half_d;
    double log2_base;
    uint64_t* mask;          // [Tp][4]
    int32_t* pos;            // [Tp]
    float2* rope_cs;         // [Tp][half_d]  (cos, sin)
    uint8_t* anc;            // [Tp][FV_CANON_DEPTH + 1]: node i's ancestor at depth d, for nodes no deeper than that (or null)
};

#ifndef FV_TS
#define FV_TS(k)   // tuning aid: a stand-alone timing harness defines this to record a time stamp
#endif
#ifndef FV_PH
#define FV_PH_DECL   // tuning aid: per-phase cycle sums inside a pipeline stage
#define FV_PH(k)
#define FV_PH_END
#endif

// one workgroup (`blk`) per four rows: their ancestor masks (a chain of dependent reads each, from LDS: out of memory 256 rows of a
// prompt took 25 us) and their rows of the rotary table (double-precision sincos, one or two entries per thread)
// (The first nodes that follow each other -- all rows of a prompt, the root tokens of a tree -- need no walk: the set of node j among them is 0..j.  The
// last of 256 prompt rows took 255 reads of LDS one after the other, 37 us a launch.)
__device__ __forceinline__ void ingest_rows(const IngestArgs& a, int blk, int32_t* s_parent, int32_t* s_depth, int* s_chain) {
    const int tid = threadIdx.x;
    if (tid < a.T) {
        const int32_t p = a.tok_in[a.cap + tid], d = a.tok_in[2 * a.cap + tid];
        s_parent[tid] = p;
        s_depth[tid] = d;
        if (a.tok_out && blk == 0) {
            a.tok_out[tid] = a.tok_in[tid];
            a.tok_out[a.cap + tid] = p;
            a.tok_out[2 * a.cap + tid] = d;
        }
        if (a.unif_in && blk == 0) {
            const double ua = a.unif_in[tid], us = a.unif_in[a.cap + tid];
            a.unif_out[tid] = ua;
            a.unif_out[a.cap + tid] = us;
        }
    }
    if (tid == 0) *s_chain = a.T;
    __syncthreads();
    if (tid < a.T && s_parent[tid] != tid - 1) atomicMin(s_chain, tid);
    __syncthreads();
    const int chain = *s_chain;   // nodes 0 .. chain - 1 each follow the one before
    const int t0 = blk * 4, t1 = (t0 + 4 < a.Tp) ? t0 + 4 : a.Tp;
    for (int i = t0 + tid; i < t1; i += 256) {
        uint64_t m[4] = {0, 0, 0, 0};
        int p = 0;
        if (i < a.T) {
            int j = i, guard = 0;
            const bool by_depth = a.anc && s_depth[i] <= FV_CANON_DEPTH;
            while (j >= 0 && guard++ < FV_MAX_TREE) {   // host validated parent[j] < j; guard bounds the walk anyway
#pragma unroll
                for (int w = 0; w < 4; ++w) m[w] |= (j >> 6) == w ? 1ull << (j & 63) : 0ull;
                if (by_depth && s_depth[j] >= 0 && s_depth[j] <= FV_CANON_DEPTH) a.anc[i * (FV_CANON_DEPTH + 1) + s_depth[j]] = (uint8_t)j;
                if (!by_depth && j < chain) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) m[w] |= j + 1 >= 64 * (w + 1) ? ~0ull : j + 1 > 64 * w ? (1ull << (j + 1 - 64 * w)) - 1ull : 0ull;
                    break;
                }
                j = s_parent[j];
            }
            p = a.L + s_depth[i];
        }
        for (int w = 0; w < 4; ++w) a.mask[i * 4 + w] = m[w];
        a.pos[i] = p;
    }
    const int n = t1 * a.half_d;
    for (int e = t0 * a.half_d + tid; e < n; e += 256) {
        const int t = e / a.half_d, i = e % a.half_d;
        const int p = (t < a.T) ? a.L + s_depth[t] : 0;
        // angle = pos * base^(-2i/d), d = 2*half_d
        const double inv_freq = exp2(-(double)i / (double)a.half_d * a.log2_base);
        double s, c;
        sincos((double)p * inv_freq, &s, &c);
        a.rope_cs[e] = make_float2((float)c, (float)s);
    }
}

// Prompt rows: a chain.  Positions and rotary rows of Tp rows from slot L on; the masks of one piece of 256 rows, which are
// those of every piece.  (ingest_rows would walk up to 255 parents per row.)
struct PromptIngestArgs { int T, Tp, L, half_d; double log2_base; uint64_t* mask; float2* rope_cs; };
// (workgroups behind the Tp / 4 of the rows clear padding)
static __global__ __launch_bounds__(256) void k_ingest_prompt(PromptIngestArgs a, PadArgs pa) {
    if ((int)blockIdx.x >= a.Tp / 4) { clear_pads(pa, (blockIdx.x - a.Tp / 4) * 256 + threadIdx.x); return; }
    const int t0 = blockIdx.x * 4, tid = threadIdx.x;
    if (t0 < 256 && tid < 16) {
        const int i = t0 + (tid >> 2), w = tid & 3, n = i + 1 - 64 * w;   // row i sees rows 0..i
        a.mask[i * 4 + w] = n <= 0 ? 0ull : n >= 64 ? ~0ull : (1ull << n) - 1ull;
    }
    for (int e = t0 * a.half_d + tid; e < (t0 + 4) * a.half_d; e += 256) {
        const int t = e / a.half_d, i = e % a.half_d;
        if (t >= a.Tp) break;
        const int p = (t < a.T) ? a.L + t : 0;
        const double inv_freq = exp2(-(double)i / (double)a.half_d * a.log2_base);
        double s, c;
        sincos((double)p * inv_freq, &s, &c);
        a.rope_cs[e] = make_float2((float)c, (float)s);
    }
}

// The last rows of a prompt that went through the layers with the others: residual stream, GEMM input and statistics of rows
// r0 .. r0+T-1 from the prompt's buffers (ld rows) into a step's (Tp rows; rows beyond T zero).  One workgroup per strip.
struct SliceArgs { const float4* x; const char* xb; const float* ssq; float4* x_out; char* xb_out; float* ssq_out; int r0, T, Tp, ld; };
template <typename EL>
static __global__ __launch_bounds__(256) void k_prompt_slice(SliceArgs a) {
    const int s = blockIdx.x, t = threadIdx.x;
    if (t >= a.Tp) return;
    const bool real = t < a.T;
    const int r = a.r0 + (real ? t : 0);
    const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 8; ++q) a.x_out[(size_t)(s * 8 + q) * a.Tp + t] = real ? a.x[(size_t)(s * 8 + q) * a.ld + r] : z4;
    constexpr int NV = 32 / Tr<EL>::E;   // 16-byte vectors of the GEMM input per strip
#pragma unroll
    for (int q = 0; q < NV; ++q) ((float4*)a.xb_out)[(size_t)(s * NV + q) * a.Tp + t] = real ? ((const float4*)a.xb)[(size_t)(s * NV + q) * a.ld + r] : z4;
    a.ssq_out[(size_t)s * a.Tp + t] = real ? a.ssq[(size_t)s * a.ld + r] : 0.f;
}

// RMSNorm factor of every row from the per-strip sums of squares, 64 rows per workgroup
struct RinvArgs { const float* ssq; float* rinv; int n_ssq, ld; float inv_h, eps; };
static __global__ __launch_bounds__(256) void k_rinv(RinvArgs a) {
    __shared__ float red[256];
    const int tid = threadIdx.x, t = blockIdx.x * 64 + (tid & 63), sl = tid >> 6;
    float s = 0.f;
#pragma unroll 8
    for (int i = sl; i < a.n_ssq; i += 4) s += a.ssq[(size_t)i * a.ld + t];
    red[tid] = s;
    __syncthreads();
    if (tid < 64) a.rinv[t] = rsqrtf((red[tid] + red[tid + 64] + red[tid + 128] + red[tid + 192]) * a.inv_h + a.eps);
}

// ============================================================================ embed
// x[:, t] = E[tok[t]];  also emits the first GEMM's input  xb = x * gain  (un-normalised;
// the RMSNorm scale 1/sqrt(mean(x^2)+eps) is applied to the GEMM result instead, it is a
// per-token factor) and the per-strip partial sums of squares.
struct EmbedArgs {
    const void* table;       // [V][h]
    const int32_t* tok;      // [cap]
    const float* gain;       // [h]
    float* x;                // [h/4][Tp][4]
    void* xb;                // vector-major [h/E][Tp][E]
    float* ssq_part;         // [h/32][Tp]
    int h, T, Tp;
};

// 32 features (strip s) of row t.  All that is read is asked for before anything is stored: the buffers could overlap for all the compiler knows, and
// with a load behind every store a strip took eight trips to memory (2000 rows of a prompt 44 us, the start of a step 6.7).
template <typename EL>
__device__ __forceinline__ void embed_strip(const EmbedArgs& a, int s, int t) {
    constexpr int E = Tr<EL>::E, NV = 32 / E;   // 16-byte vectors of a strip (rows are whole ones: h is a multiple of 64)
    uint4 raw[NV];
    float4 gn[8];
    const uint4* const row = (const uint4*)a.table + ((size_t)(t < a.T ? a.tok[t] : 0) * a.h + s * 32) / E;
#pragma unroll
    for (int k = 0; k < NV; ++k) raw[k] = t < a.T ? row[k] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int q = 0; q < 8; ++q) gn[q] = *(const float4*)(a.gain + s * 32 + q * 4);
    float ssq = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int f0 = s * 32 + q * 4;
        float v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = Tr<EL>::at(raw[q * 4 / E], (q * 4 + c) % E);
        ((float4*)a.x)[(size_t)(f0 >> 2) * a.Tp + t] = make_float4(v[0], v[1], v[2], v[3]);
        store4_act<EL>(a.xb, a.Tp, f0, t, v[0] * gn[q].x, v[1] * gn[q].y, v[2] * gn[q].z, v[3] * gn[q].w);
        ssq += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    }
    a.ssq_part[(size_t)s * a.Tp + t] = ssq;
}

// prompt rows: grid (h / 32, Tp / 256)
template <typename EL>
__global__ __launch_bounds__(256) void k_embed(EmbedArgs a) { embed_strip<EL>(a, blockIdx.x, blockIdx.y * 256 + threadIdx.x); }

// The start of a step, ingest and embedding side by side in one launch (they do not depend on each other): the first n_embed
// workgroups take 256 / Tp strips each, the next Tp / 4 four rows, the others clear padding.  Tp is 32, 64, 128 or 256.
template <typename EL>
__global__ __launch_bounds__(256) void k_begin(IngestArgs ia, EmbedArgs ea, int n_embed, PadArgs pa) {
    __shared__ int32_t s_parent[FV_MAX_TREE], s_depth[FV_MAX_TREE];
    __shared__ int s_chain;
    if ((int)blockIdx.x < n_embed) {
        const int s = blockIdx.x * (256 / ea.Tp) + threadIdx.x / ea.Tp;
        if (s < ea.h / 32) embed_strip<EL>(ea, s, threadIdx.x % ea.Tp);
    } else if ((int)blockIdx.x < n_embed + ia.Tp / 4) {
        ingest_rows(ia, blockIdx.x - n_embed, s_parent, s_depth, &s_chain);
    } else {
        clear_pads(pa, (blockIdx.x - n_embed - ia.Tp / 4) * 256 + threadIdx.x);
    }
}

// ============================================================================ skinny GEMM
// Y^T[N, Tp] = W[N, K] * X^T[K, Tp] with T = 16..256 tokens: the weights are streamed
// once from HBM, the activations come from L2 through LDS.  The (row-group x K-batch)
// space is cut into G equal contiguous ranges, one per workgroup (stream-K), so all CUs
// stream the same number of bytes whatever N and K are.  A workgroup is R wavefronts;
// wavefront w owns strip w of the row group and all of them share the X chunk in LDS.
// Each range piece that lies in one row group is a "segment".  A segment that covers the
// whole K range goes straight from registers to the epilogue; otherwise its fp32
// accumulators go to `part`, the workgroup takes a ticket on the row group's counter, and
// the workgroup that draws the last ticket sums all segments of the group in ascending
// workgroup order (so the result does not depend on who arrives last) and runs the epilogue.
enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LOGITS = 3, EPI_HEAD = 4 };

// n 32-bit words to zero (a template so that every translation unit may hold it)
template <int UNUSED>
__global__ void k_zero_words(uint32_t* p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

struct GemmArgs {
    const uint4* Wt;     // tiled weights [NG*R strips][NB][FRAGS][64] x 16 B
    const uint4* X;      // vector-major [NB*16][Tp] x 16 B
    const uint4* zeros;  // 32 KiB of zeros (what the direct kernels' padded stages load)
    float* part;         // partial tiles, fp32: [G][segmax][tiles of the kernel][1024]
    unsigned part_bytes; // size of that area (the 128-bit exchange addresses it through a bounds-checked buffer descriptor)
    int* tickets;        // [NG], zero on entry, left zero on exit (shared-activation kernel; the direct kernels draw no tickets)
    // Direct / paired kernels (fv_gemm_direct.hpp): the partial area is all zeros at the start of a launch and
    // left all zeros; a stored partial value carries `mark` in its lowest mantissa bit (1; 0 only in the host's
    // test of the time-out).  spin_limit: re-reads of a tile that has not arrived before the finishing
    // workgroup gives up, stores 1 to *fault and carries on with what it has.
    unsigned mark, spin_limit;
    unsigned* fault;
    int NG, NB, G, segmax;
    int aligned;         // direct kernels: workgroup ranges end on row-group boundaries (no partial tiles)
    // the split: workgroup w starts at unit per * w + rem * w / G of the (row group, K stage) space (aligned: at that row group)
    unsigned per, rem;
    Div div_G, div_NB;
    // stream-K split, precomputed on the host: range start of every workgroup (G+1 entries), its
    // first row group, and the first / last contributing workgroup of every row group
    const int* tab_u0; const int* tab_g0; const int* tab_cf; const int* tab_cl;
    // Deferred reduction (shared-activation kernel, 128 / 256 tokens): a segment that does not cover
    // the whole K range only stores its partial tiles, and k_gemm_fix, launched right behind, reduces
    // the n_fix row groups that have several contributors with one wavefront per tile.
    int defer, n_fix;
    const int4* fix_groups;  // [n_fix] row groups with more than one contributor: (group, first and last contributor, the first one's segment index)
    float* rinv_out;         // [Tp] RMSNorm factors handed from k_gemm to k_gemm_fix
    int T, n_strips;     // real tokens; strips that carry real rows
    // RMSNorm statistics of the input (QKV, SWIGLU, LOGITS): rinv[t] = rsqrt(sum_s ssq_in[s][t] / h + eps)
    const float* ssq_in; // [n_ssq][Tp]
    int n_ssq;
    float inv_h, eps;
    // EPI_QKV: rotate q and k, write q (vector-major), k and v into the cache at slot L + t.
    // bf16: q is kept as two bf16 tensors, q_out + q_lo_out (the second holds what the first lost to
    // rounding), so that the scores see q at about 16 mantissa bits: the attention kernel has matrix
    // cycles to spare, and rounding q to one bf16 moved the logits of a 32-layer model as much as the
    // whole K cache's rounding does.
    void* q_out;
    void* q_lo_out;
    void* kcache;        // this layer's K slabs [Hkv][S_pad*D]
    void* vcache;
    const float2* rope_cs;   // [Tp][D/2]
    int Hq, Hkv, L, S_pad;
    // EPI_RESID: x = x_in + y (x_in may be x); xb = x * gain_next; partial sums of squares of the new x
    const float* x_in;
    float* x;
    void* xb;
    const float* gain_next;
    float* ssq_out;      // [n_strips][Tp]
    // EPI_SWIGLU: act = silu(gate) * up
    void* act;
    // EPI_LOGITS
    // EPI_HEAD (a drafter's long commit): logits of which few rows are wanted.  Row L + i goes to row i, row L - Hq + j to row FV_MAX_TREE + j,
    // the rows before those nowhere; a value of any row below T and any of the first Hkv tokens that is not finite sets *tickets to 1.
    float* logits;       // [Tp][Vpad]
    int Vpad;
    int ld;              // ring kernel over a prompt: rows of the activation buffers (a multiple of 256)
};

// First unit of workgroup w's range (w = G: the end)
__device__ __forceinline__ int split_unit(const GemmArgs& a, int w) {
    const unsigned x = a.per * (unsigned)w + a.rem * (unsigned)w / a.div_G;
    return (int)(a.aligned ? x * (unsigned)a.NB : x);
}
// Asks for all of a product's arguments at once.  Read where they are used they come a cache line at a time, each a trip to memory that the next waits for.
__device__ __forceinline__ void request_args(const GemmArgs& a) {
    asm volatile("" ::"s"(a.Wt), "s"(a.zeros), "s"(a.mark), "s"(a.NG), "s"(a.aligned), "s"(a.div_NB.m), "s"(a.tab_cl), "s"(a.n_ssq), "s"(a.q_out), "s"(a.Hq), "s"(a.x),
                 "s"(a.Vpad));
}

// Epilogue of one 32-row strip x 32-token block, in accumulator layout: lane (tl, g), acc[i] is
// row 8*(i/4) + 4*g + i%4 of the strip for token tb*32 + tl.
// Inputs of an epilogue that do not depend on the GEMM result.  A caller that has to wait for
// something else first (the partial-tile exchange) requests them before that wait and hands them in.
//   EPI_RESID: x = the residual rows, gain = the next norm's gains of this lane's 16 outputs
//   EPI_QKV (q and k strips): x[2*pr], x[2*pr+1] = the four (cos, sin) pairs of rotary indices
//              16*j + 8*pr + 4*g .. +3 at this lane's token
struct EpiPre { float4 x[4], gain[4]; };
typedef EpiPre ResidPre;
__device__ __forceinline__ void resid_preload(const GemmArgs& a, int Tp, int strip, int tb, int lane, EpiPre& p) {
    const int t = tb * 32 + (lane & 31), g = lane >> 5;
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
        const int f0 = strip * 32 + 8 * blk + 4 * g;
        p.x[blk] = ((const float4*)a.x_in)[(size_t)(f0 >> 2) * Tp + t];
        p.gain[blk] = *(const float4*)(a.gain_next + f0);
    }
}
template <int D>
__device__ __forceinline__ bool rope_preload(const GemmArgs& a, int strip, int tb, int lane, EpiPre& p) {
    constexpr int SPH = D / 32;
    const int t = tb * 32 + (lane & 31), g = lane >> 5, j = strip % SPH;
    if (strip / SPH >= a.Hq + a.Hkv) return false;   // a v strip: no rotation
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
        const float4* cp = (const float4*)(a.rope_cs + (size_t)t * (D / 2) + 16 * j + 8 * pr + 4 * g);
        p.x[2 * pr] = cp[0];
        p.x[2 * pr + 1] = cp[1];
    }
    return true;
}

// IN_ORDER: the squares are added in a written order, not in one that the compiler picks for each kernel.  The direct, paired and small forms have it: steps of up
// to 64 rows take one or another by their row count, and a node's bits must not depend on that.
template <typename EL, int D, int EPI, bool IN_ORDER = false>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, int Tp, int strip, int tb, int lane, float (&acc)[16],
                                              const float* rinv_lds, const EpiPre& pre, bool have_pre) {
    const int tl = lane & 31, g = lane >> 5;
    const int t = tb * 32 + tl;
    if constexpr (EPI == EPI_RESID) {
        float ssq = 0.f;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
            const int f0 = strip * 32 + 8 * blk + 4 * g;
            float4 xv = pre.x[blk], gn = pre.gain[blk];
            if (!have_pre) { xv = ((const float4*)a.x_in)[(size_t)(f0 >> 2) * Tp + t]; gn = *(const float4*)(a.gain_next + f0); }
            xv.x += acc[4 * blk]; xv.y += acc[4 * blk + 1]; xv.z += acc[4 * blk + 2]; xv.w += acc[4 * blk + 3];
            st_f4((float4*)a.x + (size_t)(f0 >> 2) * Tp + t, xv);
            store4_act<EL>(a.xb, Tp, f0, t, xv.x * gn.x, xv.y * gn.y, xv.z * gn.z, xv.w * gn.w);
            if constexpr (IN_ORDER) ssq += fmaf(xv.w, xv.w, fmaf(xv.z, xv.z, fmaf(xv.y, xv.y, xv.x * xv.x)));
            else ssq += xv.x * xv.x + xv.y * xv.y + xv.z * xv.z + xv.w * xv.w;
        }
        ssq += __shfl_xor(ssq, 32);
        if (g == 0) st_f32(a.ssq_out + (size_t)strip * Tp + t, ssq);
    } else {
        const float rs = rinv_lds[t];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] *= rs;
        if constexpr (EPI == EPI_LOGITS) {
#pragma unroll
            for (int blk = 0; blk < 4; ++blk) {
                const int f0 = strip * 32 + 8 * blk + 4 * g;
                st_f4((float4*)(a.logits + (size_t)t * a.Vpad + f0),
                           make_float4(acc[4 * blk], acc[4 * blk + 1], acc[4 * blk + 2], acc[4 * blk + 3]));
            }
        } else if constexpr (EPI == EPI_HEAD) {
            bool bad = false;
            const int row = t >= a.L ? t - a.L : t >= a.L - a.Hq ? FV_MAX_TREE + t - (a.L - a.Hq) : -1;
#pragma unroll
            for (int blk = 0; blk < 4; ++blk) {
                const int f0 = strip * 32 + 8 * blk + 4 * g;
#pragma unroll
                for (int c = 0; c < 4; ++c) bad = bad || (f0 + c < a.Hkv && !(__builtin_fabsf(acc[4 * blk + c]) < INFINITY));
                if (t < a.T && row >= 0)
                    st_f4((float4*)(a.logits + (size_t)row * a.Vpad + f0), make_float4(acc[4 * blk], acc[4 * blk + 1], acc[4 * blk + 2], acc[4 * blk + 3]));
            }
            if (bad && t < a.T) *a.tickets = 1;
        } else if constexpr (EPI == EPI_SWIGLU) {
            // strip covers activation features [16*strip, 16*strip+16): accumulator blocks 0,2 are
            // gate rows, blocks 1,3 the matching up rows
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                float o[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float gt = acc[8 * pr + c], up = acc[8 * pr + 4 + c];
                    o[c] = gt / (1.f + __expf(-gt)) * up;
                }
                store4_act<EL>(a.act, Tp, 16 * strip + 8 * pr + 4 * g, t, o[0], o[1], o[2], o[3]);
            }
        } else {  // EPI_QKV
            constexpr int SPH = D / 32;   // strips per head
            const int head = strip / SPH, j = strip % SPH;
            if (head < a.Hq + a.Hkv) {
                // q or k head: blocks (0,1) and (2,3) are rotary pairs (i, i + D/2)
                float lo_v[2][4], hi_v[2][4];
#pragma unroll
                for (int pr = 0; pr < 2; ++pr) {
                    // (cos, sin) of indices 16*j + 8*pr + 4*g + c in the first half of the head, c = 0..3
                    float4 c01 = pre.x[2 * pr], c23 = pre.x[2 * pr + 1];
                    if (!have_pre) {
                        const float4* cp = (const float4*)(a.rope_cs + (size_t)t * (D / 2) + 16 * j + 8 * pr + 4 * g);
                        c01 = cp[0]; c23 = cp[1];
                    }
                    const float co[4] = {c01.x, c01.z, c23.x, c23.z}, si[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float x1 = acc[8 * pr + c], x2 = acc[8 * pr + 4 + c];
                        lo_v[pr][c] = x1 * co[c] - x2 * si[c];
                        hi_v[pr][c] = x2 * co[c] + x1 * si[c];
                    }
                }
                if (head < a.Hq) {
#pragma unroll
                    for (int pr = 0; pr < 2; ++pr) {
                        const int f1 = head * D + 16 * j + 8 * pr + 4 * g;
                        store4_act<EL>(a.q_out, Tp, f1, t, lo_v[pr][0], lo_v[pr][1], lo_v[pr][2], lo_v[pr][3]);
                        store4_act<EL>(a.q_out, Tp, f1 + D / 2, t, hi_v[pr][0], hi_v[pr][1], hi_v[pr][2], hi_v[pr][3]);
                        if constexpr (Tr<EL>::E == 8) {
                            store4_act<EL>(a.q_lo_out, Tp, f1, t, bf16_residual(lo_v[pr][0]), bf16_residual(lo_v[pr][1]),
                                           bf16_residual(lo_v[pr][2]), bf16_residual(lo_v[pr][3]));
                            store4_act<EL>(a.q_lo_out, Tp, f1 + D / 2, t, bf16_residual(hi_v[pr][0]), bf16_residual(hi_v[pr][1]),
                                           bf16_residual(hi_v[pr][2]), bf16_residual(hi_v[pr][3]));
                        }
                    }
                } else if (t < a.T) {
                    const int kh = head - a.Hq;
                    char* slab = (char*)a.kcache + (size_t)kh * a.S_pad * D * Tr<EL>::ESZ;
                    const int pos = a.L + t;   // cache SLOT of tree node t (its rotary position is L + depth)
                    // four consecutive features of one position are contiguous in the slab (they lie in
                    // one 2E-feature fragment row): one 8- or 16-byte store each
#pragma unroll
                    for (int pr = 0; pr < 2; ++pr) {
                        const int f1 = 16 * j + 8 * pr + 4 * g;
                        st_cache4<EL>(slab, kcache_index<EL, D>(pos, f1), lo_v[pr]);
                        st_cache4<EL>(slab, kcache_index<EL, D>(pos, f1 + D / 2), hi_v[pr]);
                    }
                }
            } else if (t < a.T) {
                const int kh = head - a.Hq - a.Hkv;
                char* slab = (char*)a.vcache + (size_t)kh * a.S_pad * D * Tr<EL>::ESZ;
                const int pos = a.L + t;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int f = 32 * j + 8 * (i >> 2) + 4 * g + (i & 3);
                    st_elem<EL>(slab, vcache_index<EL, D>(pos, f), acc[i]);
                }
            }
        }
    }
}

template <typename EL, int D, int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, int Tp, int strip, int tb, int lane, float (&acc)[16],
                                              const float* rinv_lds) {
    EpiPre none;   // never read: have_pre = false
    gemm_epilogue<EL, D, EPI>(a, Tp, strip, tb, lane, acc, rinv_lds, none, false);
}

// One stage of the shared-activation GEMM for one wavefront: FV_FRAGS weight fragments (registers)
// times TB activation tiles each (LDS).  The B tiles of fragment f+1 are requested before the
// MFMAs of fragment f are issued, so an LDS read has TB MFMAs (32 cycles each) to land in;
// between_frags(f) runs after the MFMAs of fragment f have been issued -- the kernel puts a slice
// of the next stages' global loads there, so that the texture-address path works through them
// while the matrix cores are busy instead of after them.
template <typename EL, int TB, typename Between>
__device__ __forceinline__ void gemm_compute(const uint4 (&w)[FV_FRAGS], const uint4* __restrict__ xl,
                                             floatx16 (&acc)[TB], int lane, Between&& between_frags) {
    constexpr int Tp = TB * 32;
    const int t = lane & 31, g = lane >> 5;
    const uint4* xb = xl + g * Tp + t;
    uint4 b[2][TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) b[0][tb] = xb[tb * 32];
#pragma unroll
    for (int f = 0; f < FV_FRAGS; ++f) {
        if (f + 1 < FV_FRAGS) {
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) b[(f + 1) & 1][tb] = xb[2 * (f + 1) * Tp + tb * 32];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[tb] = Tr<EL>::mma(w[f], b[f & 1][tb], acc[tb]);
        __builtin_amdgcn_sched_barrier(0);
        between_frags(f);
        __builtin_amdgcn_sched_barrier(0);
    }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // a 16-byte register quad as a first-class value

template <int N, int STRIDE>
__device__ __forceinline__ void ld_vec(uint4 (&dst)[N], const uint4* __restrict__ src) {
#pragma unroll
    for (int v = 0; v < N; ++v) dst[v] = src[v * STRIDE];
}
template <int N, int STRIDE>
__device__ __forceinline__ void ld_x(u32x4 (&dst)[N], const uint4* __restrict__ src) {
#pragma unroll
    for (int v = 0; v < N; ++v) dst[v] = *(const u32x4*)(src + v * STRIDE);
}
template <int N, int STRIDE>
__device__ __forceinline__ void st_lds(uint4* dst, const u32x4 (&src)[N]) {
#pragma unroll
    for (int v = 0; v < N; ++v) *(u32x4*)(dst + v * STRIDE) = src[v];
}
template <int TB>
__device__ __forceinline__ void zero_acc(floatx16 (&acc)[TB]) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[tb][i] = 0.f;
}

// Ends one segment (a run of K batches of one row group): either straight to the epilogue
// (the segment covered the whole K range) or partials + ticket + last-arriver reduction.
//
// Partial tiles cross XCDs, whose L2s are not coherent with each other, so they are written
// and read with the agent-scope cache policy (write-through stores, loads that do not hit a
// stale line) and no whole-L2 write-back or invalidate is needed.  They move as 128-bit
// accesses (layout per tile [4 register quads][64 lanes][4 floats], 1 KiB per wavefront
// access): a wavefront can have 64 memory operations in flight, and with one-register
// accesses that cap, not the memory system, set the pace of a reduction over many
// contributors.  The 128-bit accesses go through a raw buffer descriptor over the partial
// area, which carries the same policy bit as the agent-scope atomics and bounds-checks
// every address in hardware.
template <typename EL, int TB, int D, int EPI>
__device__ __forceinline__ void gemm_flush(const GemmArgs& a, floatx16 (&acc)[TB], int gi, int seg_batches, int seg,
                                           const float* rinv_lds, int* ticket_lds) {
    constexpr int R = FV_R;
    constexpr int Tp = TB * 32;
    constexpr int TG = TB < 4 ? TB : 4;   // tiles handled together: their loads are in flight at the same time
    // early epilogue inputs; not for the rotary epilogue at 256 tokens, where their registers are spilled
    constexpr bool PRE = (EPI == EPI_RESID || (EPI == EPI_QKV && TB <= 4));
    constexpr int SC1 = 16;               // cache-policy operand of the buffer accesses: agent scope
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int strip = gi * R + wave;
    // what the epilogues of tiles t0 .. t0+TG-1 read besides the GEMM result, requested early
    auto preload = [&](int t0, EpiPre (&pre)[TG]) -> bool {
        bool have = false;
        if constexpr (EPI == EPI_RESID) {
#pragma unroll
            for (int tb = 0; tb < TG; ++tb) resid_preload(a, Tp, strip, t0 + tb, lane, pre[tb]);
            have = true;
        } else if constexpr (EPI == EPI_QKV) {
#pragma unroll
            for (int tb = 0; tb < TG; ++tb) have = rope_preload<D>(a, strip, t0 + tb, lane, pre[tb]);
        }
        return have;
    };
    if (seg_batches == a.NB) {
        // the whole K range of this row group was ours: no partials, no ticket
        if (strip < a.n_strips) {
#pragma unroll
            for (int t0 = 0; t0 < TB; t0 += TG) {
                EpiPre pre[TG];
                const bool have = PRE && preload(t0, pre);
#pragma unroll
                for (int tb = 0; tb < TG; ++tb) {
                    float r[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) r[i] = acc[t0 + tb][i];
                    gemm_epilogue<EL, D, EPI>(a, Tp, strip, t0 + tb, lane, r, rinv_lds, pre[tb], have);
                }
            }
        }
        return;
    }
    const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc((void*)a.part, 0, (int)a.part_bytes, 0x00020000);   // raw, 32-bit data format
    auto tile_ofs = [&](int wg, int sg, int tb) -> unsigned {   // byte offset of this lane's first quad of a tile
        return ((unsigned)(((wg * a.segmax + sg) * R + wave) * TB + tb) * 1024u + (unsigned)lane * 4u) * 4u;
    };
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        const unsigned o = tile_ofs((int)blockIdx.x, seg, tb);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32x4 v;
            v.x = __float_as_uint(acc[tb][4 * q]); v.y = __float_as_uint(acc[tb][4 * q + 1]);
            v.z = __float_as_uint(acc[tb][4 * q + 2]); v.w = __float_as_uint(acc[tb][4 * q + 3]);
            __builtin_amdgcn_raw_buffer_store_b128(v, prs, o + q * 1024u, 0, SC1);
        }
    }
    if (a.defer) return;   // reduced by k_gemm_fix after this launch (the launch boundary orders the two)
    // contributors of row group gi: workgroups c_first..c_last (each has a non-empty range); the
    // ranges are contiguous, so every contributor but the first starts inside the group (its
    // segment index for it is 0)
    const int c_first = a.tab_cf[gi], c_last = a.tab_cl[gi];
    const int seg_first = gi - a.tab_g0[c_first];
    // Release: the payload was stored write-through, so it is enough that every lane's stores
    // have been acknowledged (vmcnt(0): on this target stores count in vmcnt) before the
    // ticket is drawn.
    handoff_release();
    FV_TS(3)
    __syncthreads();
    if (tid == 0)
        *ticket_lds = __hip_atomic_fetch_add(&a.tickets[gi], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    handoff_acquire();
    FV_TS(4)
    const bool last = (*ticket_lds == c_last - c_first);
    if (last) {
        // every other contributor's ticket, hence its acknowledged stores, precede ours
        if (tid == 0) __hip_atomic_store(&a.tickets[gi], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
        if (strip < a.n_strips) {
            // KC contributors x TG tiles (up to 32 KiB per wavefront) are in flight at a time; the
            // sum runs in ascending contributor order, so it does not depend on who arrived last
            constexpr int KC = TG <= 2 ? 4 : (TB <= 4 ? 2 : 1);   // at 256 tokens the activation staging registers leave room for one
#pragma unroll
            for (int t0 = 0; t0 < TB; t0 += TG) {
                EpiPre pre[TG];
                const bool have = PRE && preload(t0, pre);
                float r[TG][16];
#pragma unroll
                for (int tb = 0; tb < TG; ++tb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) r[tb][i] = 0.f;
                for (int c0 = c_first; c0 <= c_last; c0 += KC) {
                    u32x4 v[KC][TG][4];
#pragma unroll
                    for (int k = 0; k < KC; ++k) {
                        const int c = (c0 + k <= c_last) ? c0 + k : c_last;
                        const unsigned o = tile_ofs(c, (c == c_first) ? seg_first : 0, t0);
#pragma unroll
                        for (int tb = 0; tb < TG; ++tb)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                v[k][tb][q] = __builtin_amdgcn_raw_buffer_load_b128(prs, o + (tb * 4 + q) * 1024u, 0, SC1);
                    }
#pragma unroll
                    for (int k = 0; k < KC; ++k) {
                        const float m = (c0 + k <= c_last) ? 1.f : 0.f;
#pragma unroll
                        for (int tb = 0; tb < TG; ++tb)
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                r[tb][4 * q] += m * __uint_as_float(v[k][tb][q].x);
                                r[tb][4 * q + 1] += m * __uint_as_float(v[k][tb][q].y);
                                r[tb][4 * q + 2] += m * __uint_as_float(v[k][tb][q].z);
                                r[tb][4 * q + 3] += m * __uint_as_float(v[k][tb][q].w);
                            }
                    }
                }
                if (t0 == 0) { FV_TS(5) }
#pragma unroll
                for (int tb = 0; tb < TG; ++tb) gemm_epilogue<EL, D, EPI>(a, Tp, strip, t0 + tb, lane, r[tb], rinv_lds, pre[tb], have);
            }
            FV_TS(6)
        }
    }
    __syncthreads();   // ticket_lds is reused by the next segment
}

template <typename EL, int TB, int D, int EPI>
__global__ __launch_bounds__(64 * FV_R, 1) void k_gemm(GemmArgs a) {
    extern __shared__ uint4 lds[];
    constexpr int R = FV_R;
    constexpr int Tp = TB * 32;
    constexpr int CV = Tp * 16;          // uint4 per X chunk (Tp tokens x 256 B)
    constexpr int XV = CV / (64 * R);    // uint4 per thread per chunk
    static_assert(CV % (64 * R) == 0, "chunk must divide over the workgroup");
    __shared__ float rinv_lds[Tp];
    __shared__ __attribute__((aligned(16))) float red_lds[(EPI == EPI_RESID) ? 4 : 1024];
    __shared__ int ticket_lds;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if ((int)blockIdx.x >= a.G) return;
    FV_TS(0)

    // This workgroup's units [u0, u1) of the (row group, K batch) space are one software-pipelined
    // stream: the weight tiles and the activation chunk of stage k+2 are requested while stage k is
    // multiplied (weights into the third register set, the chunk into staging registers that go to
    // the other LDS buffer one stage later), across row-group boundaries too.  Every segment (the
    // part of the range inside one row group) is padded to whole rounds of three stages; a padded
    // stage loads zeros as its activation chunk (and one weight line, finite), so the loop body has
    // no conditional, the accumulators stay in the accumulation registers, and the number of loads
    // per stage -- which the wait counts are computed from -- is fixed.
    const int u0 = split_unit(a, blockIdx.x), u1 = split_unit(a, blockIdx.x + 1);   // computed, not looked up: no extra round trip before the first load
    const int g0 = (int)((unsigned)u0 / a.div_NB);
    int nseg = 1;
    for (int e_ = (g0 + 1) * a.NB; e_ < u1; e_ += a.NB) ++nseg;
    auto segment = [&](int sgm, int& gi, int& b0, int& nb) {
        gi = g0 + sgm;
        b0 = (sgm == 0) ? u0 - g0 * a.NB : 0;
        const int rem = u1 - gi * a.NB;
        nb = (rem < a.NB ? rem : a.NB) - b0;
    };
    // weights are tiled [strip pair][half K batch][2 strips][4 frags]: this wavefront's strip is strip (wave % 2) of pair
    // gi * 2 + wave / 2; a K batch of it is two 4 KiB pieces 8 KiB apart, and batches follow each other 16 KiB apart
    const uint4* __restrict__ wbase = a.Wt + ((size_t)(wave >> 1) * (2 * a.NB) * 2 + (wave & 1)) * (4 * 64) + lane;
    const size_t group_stride = (size_t)R * a.NB * (FV_FRAGS * 64);
    const uint4* const zeros = a.zeros;

    // request position: segment rs, padded stage rj of rn3 (rn real ones), this thread's addresses
    int rs = 0, rj = 0, rn = 0, rn3 = 0;
    const uint4* wp = a.Wt;
    const uint4* xp = zeros;
    auto enter = [&](int sgm) {
        rs = sgm; rj = 0; rn = 0; rn3 = 0; wp = a.Wt; xp = zeros;
        if (rs < nseg) {
            int gi, b0, nb;
            segment(rs, gi, b0, nb);
            rn = nb; rn3 = (nb + 2) / 3 * 3;
            wp = wbase + (size_t)gi * group_stride + (size_t)b0 * (2 * FV_FRAGS * 64);
            xp = a.X + (size_t)b0 * CV + tid;
        }
    };
    auto advance = [&]() {
        ++rj; wp += 2 * FV_FRAGS * 64; xp += CV;
        if (rj >= rn3) enter(rs + 1);
    };
    auto load_w = [&](uint4 (&dst)[FV_FRAGS]) {
        const bool live = rj < rn;
        const uint4* pw = live ? wp : a.Wt;
        const int st = live ? 64 : 0;
#pragma unroll
        for (int f = 0; f < FV_FRAGS; ++f) dst[f] = pw[(f < 4 ? f : f + 4) * st];
    };
    auto load_x = [&](u32x4 (&dst)[XV]) {
        const bool live = rj < rn;
        const uint4* px = live ? xp : zeros;
        const int st = live ? 64 * R : 0;
#pragma unroll
        for (int v = 0; v < XV; ++v) dst[v] = *(const u32x4*)(px + v * st);
    };
    uint4 w[3][FV_FRAGS];
    u32x4 xr[XV];
    enter(0);
    // prologue: W(0) first, so that it is in flight during the statistics below
    load_w(w[0]);
    if constexpr (EPI != EPI_RESID) {
        // RMSNorm factor of every token, while the first weight tiles are in flight.  The
        // [n_ssq][Tp] partial sums of squares are read as float4 (4 tokens) with eight
        // independent loads in flight per thread, then reduced over strip slices in LDS.
        constexpr int C4 = Tp / 4;            // float4 columns
        constexpr int SL = 256 / C4;          // strip slices
        const int col = tid % C4, sl = tid / C4;
        const float4* sp = (const float4*)a.ssq_in + col;
        float4 s4 = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int i0 = sl; i0 < a.n_ssq; i0 += 8 * SL) {
            float4 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int i = i0 + k * SL;
                v[k] = (i < a.n_ssq) ? sp[(size_t)i * C4] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) { s4.x += v[k].x; s4.y += v[k].y; s4.z += v[k].z; s4.w += v[k].w; }
        }
        ((float4*)red_lds)[sl * C4 + col] = s4;
        __syncthreads();
        if (tid < Tp) {
            float tot = 0.f;
#pragma unroll
            for (int p = 0; p < SL; ++p) tot += red_lds[p * Tp + tid];
            const float rv = rsqrtf(tot * a.inv_h + a.eps);
            rinv_lds[tid] = rv;
            if (a.defer && blockIdx.x == 0) a.rinv_out[tid] = rv;
        }
    }
    // X(0) -> LDS[0]; then X(1) and W(1) are issued in the same order as inside the loop
    // (activation chunk before weight tiles), so the loop's wait counts hold from the first stage
    load_x(xr);
    st_lds<XV, 64 * R>(lds + tid, xr);
    __builtin_amdgcn_sched_barrier(0);
    advance();   // stage 1
    load_x(xr);
    __builtin_amdgcn_sched_barrier(0);
    load_w(w[1]);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    FV_TS(1)

    FV_PH_DECL
    int par = 0;   // LDS buffer that holds the current stage's chunk
    // One pipeline stage with weight register set S; the loads it issues (stage + 2) go to set S2.
    // The chunk of stage + 1 goes from its staging registers to the other LDS buffer first (every
    // wavefront is past the barrier, so nobody reads that buffer any more); that frees the staging
    // registers, and the NLD loads of stage + 2 (activation chunk first, then weight tiles) are
    // issued in slices between the fragments of this stage's multiplication.
    constexpr int NLD = XV + FV_FRAGS;
#define FV_STAGE(S, S2)                                                                                 \
    {                                                                                                   \
        st_lds<XV, 64 * R>(lds + (par ^ 1) * CV + tid, xr);                                             \
        __builtin_amdgcn_sched_barrier(0);                                                              \
        FV_PH(1)                                                                                        \
        advance();                                                                                      \
        const bool live_ = rj < rn;                                                                     \
        const uint4* const px_ = live_ ? xp : zeros;                                                    \
        const uint4* const pw_ = live_ ? wp : a.Wt;                                                     \
        const int sx_ = live_ ? 64 * R : 0, sw_ = live_ ? 64 : 0;                                       \
        gemm_compute<EL, TB>(w[S], lds + par * CV, acc, lane, [&](int f) {                              \
            _Pragma("unroll") for (int i_ = f * NLD / FV_FRAGS; i_ < (f + 1) * NLD / FV_FRAGS; ++i_) {  \
                if (i_ < XV) xr[i_] = *(const u32x4*)(px_ + i_ * sx_);                                  \
                else w[S2][i_ - XV] = pw_[((i_ - XV) < 4 ? (i_ - XV) : (i_ - XV) + 4) * sw_];                                             \
            }                                                                                           \
        });                                                                                             \
        FV_PH(0)                                                                                        \
        __syncthreads();                                                                                \
        FV_PH(3)                                                                                        \
        par ^= 1;                                                                                       \
    }

    for (int sgm = 0; sgm < nseg; ++sgm) {
        int gi, b0, nb;
        segment(sgm, gi, b0, nb);
        const int rounds = (nb + 2) / 3;
        floatx16 acc[TB];
        zero_acc<TB>(acc);
        for (int r = 0; r < rounds; ++r) {
            FV_STAGE(0, 2)
            FV_STAGE(1, 0)
            FV_STAGE(2, 1)
        }
        FV_TS(2)
        gemm_flush<EL, TB, D, EPI>(a, acc, gi, nb, sgm, rinv_lds, &ticket_lds);
    }
    FV_TS(7)
    FV_PH_END
#undef FV_STAGE
}

// Second half of a deferred reduction: one wavefront per (row group with several contributors,
// strip, token block) tile sums the contributors' partial tiles in ascending workgroup order and
// runs the epilogue.  Spreading the tiles over the whole chip instead of leaving each row group
// to its last arriver matters at 128 / 256 tokens, where a row group's partials are 0.5-1 MiB and
// one CU pulls them in at ~60 GB/s.
template <typename EL, int TB, int D, int EPI>
__global__ __launch_bounds__(256) void k_gemm_fix(GemmArgs a) {
    constexpr int R = FV_R;
    constexpr int Tp = TB * 32;
    constexpr int SC1 = 16;
    __shared__ float rinv_lds[Tp];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if constexpr (EPI != EPI_RESID) {
        if (tid < Tp) rinv_lds[tid] = a.rinv_out[tid];
        __syncthreads();
    }
    const int tile = blockIdx.x * 4 + wave;
    if (tile >= a.n_fix * R * TB) return;
    const int4 rec = a.fix_groups[tile / (R * TB)];   // one load: nothing else stands between kernel entry and the partial loads
    const int gi = rec.x, c_first = rec.y, c_last = rec.z, seg_first = rec.w;
    const int r = (tile / TB) % R, tb = tile % TB;
    const int strip = gi * R + r;
    if (strip >= a.n_strips) return;
    EpiPre pre;
    bool have = false;
    if constexpr (EPI == EPI_RESID) { resid_preload(a, Tp, strip, tb, lane, pre); have = true; }
    if constexpr (EPI == EPI_QKV) have = rope_preload<D>(a, strip, tb, lane, pre);
    const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc((void*)a.part, 0, (int)a.part_bytes, 0x00020000);
    float acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    for (int c0 = c_first; c0 <= c_last; c0 += 4) {   // four contributors in flight, summed in ascending order
        u32x4 v[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int c = (c0 + k <= c_last) ? c0 + k : c_last;
            const unsigned o = ((unsigned)(((c * a.segmax + ((c == c_first) ? seg_first : 0)) * R + r) * TB + tb) * 1024u + (unsigned)lane * 4u) * 4u;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[k][q] = __builtin_amdgcn_raw_buffer_load_b128(prs, o + q * 1024u, 0, SC1);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float m = (c0 + k <= c_last) ? 1.f : 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc[4 * q] += m * __uint_as_float(v[k][q].x);
                acc[4 * q + 1] += m * __uint_as_float(v[k][q].y);
                acc[4 * q + 2] += m * __uint_as_float(v[k][q].z);
                acc[4 * q + 3] += m * __uint_as_float(v[k][q].w);
            }
        }
    }
    gemm_epilogue<EL, D, EPI>(a, Tp, strip, tb, lane, acc, rinv_lds, pre, have);
}

#include "fv_gemm_direct.hpp"
#include "fv_gemm_small.hpp"
#include "fv_gemm_ring.hpp"

// ============================================================================ tree attention
// For node t and query head qh: softmax over {cache slots 0..L-1} U {tree slots L+j : j in
// ancestors-or-self(t)} of q.k/sqrt(D), times V.  A workgroup handles one (query head,
// block of 32 nodes); its four wavefronts take every fourth 32-key block, keep online-softmax
// statistics, and are merged through LDS.  Scores are computed transposed (keys x nodes)
// so that each lane owns one node: the node's 256-bit ancestor set sits in registers and
// is tested per key, and the probabilities are already in B-operand order for V^T * P^T.
struct AttnArgs {
    const uint4* q;          // vector-major [Hq*D/E][Tp]
    const uint4* q_lo;       // bf16 only: the part of q that q's bf16 rounding lost (same layout)
    const uint4* kc;         // this layer's K slabs
    const uint4* vc;
    void* out;               // vector-major [Hq*D/E][Tp]
    const uint64_t* mask;    // [Tp][4]
    int Tp, T, L, Hq, Hkv, S_pad;
    int ld;                  // rows of the q and out buffers (Tp, or more when a prompt's pieces are rows of one buffer)
    int pieces;              // > 1: grid.y prompt pieces of 256 rows each, row 0 of piece j at slot L + 256 j; T counts all rows
    int TK;                  // step rows whose keys exist, slots L .. L+TK-1 (= T in a verification step; a drafting pass also sees
                             // the rows of the phase's earlier passes); the masks have no bits at or above TK
    float scale;
    // key split: every (head, node block) item is shared by `ks` workgroups, each taking a
    // contiguous run of 32-key blocks; their (max, sum, unnormalised output) triples meet in
    // `part` ([item*ks + k][D/32 * 1024 + 64] floats) behind one ticket per item
    int ks;
    float* part;
    int* tickets;
};

#define FV_ATTN_SMEM_FLOATS(D) (4 * ((D) / 32) * 64 * 16 + 8 * 32 + 4)   // [feature block][wavefront][4 quads][64 lanes][4], then maxima and sums
#define FV_ATTN_PART_FLOATS(D) (((D) / 32) * 1024 + 64)

// One (query head, block of 32 nodes) item, key part `part` of a.ks.  SHARE: two workgroups of this form fit a compute unit, so that
// one wavefront of a SIMD is at its softmax or waits for K and V while the other multiplies.  For that q, the same in all four
// wavefronts, lies in LDS (64 registers less), and a block every node sees goes without the tests.  Both forms compute the same bits.
// Over ranges of a few blocks a wavefront it loses what the way through LDS costs; attn_shares has the rule and the figures.
template <typename EL, int D, bool SHARE>
__device__ __forceinline__ void attn_body(const AttnArgs& a, int item, int part, float* smem) {
    constexpr int E = Tr<EL>::E;
    constexpr int NF = D / (2 * E);      // K frags per key block
    constexpr int NQ = 32 / (2 * E);     // V frags per (key block, 32 features)
    constexpr int DB = D / 32;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int tl = lane & 31, g = lane >> 5;
    const int TB = a.Tp >> 5;
    const int qh = item / TB, tb = item % TB;
    const int kh = qh / (a.Hq / a.Hkv);
    const int t = tb * 32 + tl;

    constexpr bool SPLIT = (E == 8);   // bf16: q and the probabilities enter the matrix cores as hi + lo pairs
    constexpr int NQF = SHARE ? 1 : NF;
    uint4 qf[NQF], qfl[SPLIT ? NQF : 1];
    if constexpr (SHARE) {
        // [fragment][hi, lo][64 lanes].  (Declared here and where it is read: outside of them it changed the other form too, whose q loads then waited for
        // one more integer division.)
        uint4* const q_lds = (uint4*)smem + lane;
        for (int fr = wave; fr < NF; fr += 4) {
            const size_t at = ((size_t)(qh * (D / E) + 2 * fr + g)) * a.ld + t;
            q_lds[(2 * fr) * 64] = a.q[at];
            if constexpr (SPLIT) q_lds[(2 * fr + 1) * 64] = a.q_lo[at];
        }
        __syncthreads();
    } else {
#pragma unroll
        for (int fr = 0; fr < NF; ++fr) qf[fr] = a.q[((size_t)(qh * (D / E) + 2 * fr + g)) * a.ld + t];
        if constexpr (SPLIT) {
#pragma unroll
            for (int fr = 0; fr < NF; ++fr) qfl[fr] = a.q_lo[((size_t)(qh * (D / E) + 2 * fr + g)) * a.ld + t];
        }
    }
    uint64_t mk[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) mk[w] = (t < a.T) ? a.mask[t * 4 + w] : 0ull;

    const size_t slab_vecs = (size_t)a.S_pad * D / E;
    const uint4* kslab = a.kc + (size_t)kh * slab_vecs;
    const uint4* vslab = a.vc + (size_t)kh * slab_vecs;

    floatx16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    float m_run = -1e30f, l_run = 0.f;

    const int n_keys = a.L + a.TK;
    const int nkb = (n_keys + 31) >> 5;
    const int kb_lo = nkb * part / a.ks, kb_hi = nkb * (part + 1) / a.ks;   // this workgroup's key blocks
    const int lidx = tl * 2 + g;   // position of this lane's 16 bytes inside a 1 KiB tile
    auto load_k = [&](uint4 (&kt)[NF], int kb) {
        const uint4* kp = kslab + (size_t)kb * NF * 64 + lidx;
#pragma unroll
        for (int fr = 0; fr < NF; ++fr) kt[fr] = kp[fr * 64];
    };
    auto load_v = [&](uint4 (&vt)[DB * NQ], int kb) {
        const uint4* vp = vslab + (size_t)kb * DB * NQ * 64 + lidx;
#pragma unroll
        for (int j = 0; j < DB * NQ; ++j) vt[j] = vp[j * 64];
    };
    auto use_block = [&](uint4 (&kt)[NF], const uint4 (&vt)[DB * NQ], int kb, int kb_next) {
        // two accumulation chains (a dependent MFMA waits ~50 cycles for its predecessor, two
        // interleaved chains issue back to back), added at the end
        floatx16 s, s1;
#pragma unroll
        for (int i = 0; i < 16; ++i) { s[i] = 0.f; s1[i] = 0.f; }
        if constexpr (SHARE) {
            const uint4* const q_lds = (const uint4*)smem + lane;
            uint4 qb[2][4];   // a pair of fragments, hi and lo, read while the pair before multiplies
            auto read_q = [&](int fr, uint4 (&d)[4]) {
#pragma unroll
                for (int k = 0; k < 4; ++k) if (SPLIT || !(k & 1)) d[k] = q_lds[(2 * fr + k) * 64];
            };
            read_q(0, qb[0]);
#pragma unroll
            for (int fr = 0; fr < NF; fr += 2) {
                __builtin_amdgcn_sched_barrier(0);
                if (fr + 2 < NF) read_q(fr + 2, qb[(fr / 2 + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                const uint4 (&d)[4] = qb[(fr / 2) & 1];
                s = Tr<EL>::mma(kt[fr], d[0], s);
                s1 = Tr<EL>::mma(kt[fr + 1], d[2], s1);
                if constexpr (SPLIT) {
                    s = Tr<EL>::mma(kt[fr], d[1], s);
                    s1 = Tr<EL>::mma(kt[fr + 1], d[3], s1);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
            for (int fr = 0; fr < NF; fr += 2) {
                s = Tr<EL>::mma(kt[fr], qf[fr], s);
                s1 = Tr<EL>::mma(kt[fr + 1], qf[fr + 1], s1);
                if constexpr (SPLIT) {
                    s = Tr<EL>::mma(kt[fr], qfl[fr], s);
                    s1 = Tr<EL>::mma(kt[fr + 1], qfl[fr + 1], s1);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        load_k(kt, kb_next);   // into the registers that the products have just read
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] += s1[i];

        // Visibility of the block's 32 keys for this lane's node as one 32-bit word (bit j: key
        // kb*32 + j): prefix keys are visible to every node, a tree key n only if bit n of the node's
        // ancestor mask is set (the mask has no bits at or above T).  The block's offset into the
        // tree, n0, is the same for the whole wavefront, so the window is cut out of the 256-bit
        // mask with uniform shifts and no per-element branch.
        uint32_t vbits = 0xffffffffu;
        const int n0 = kb * 32 - a.L;   // tree index of the block's first key
        if (n0 > -32) {
            uint32_t win;
            if (n0 < 0) {
                win = ((1u << (-n0)) - 1u) | ((uint32_t)mk[0] << (-n0));
            } else {
                const int w = n0 >> 6, sh = n0 & 63;
                const uint64_t lo = (w == 0) ? mk[0] : (w == 1) ? mk[1] : (w == 2) ? mk[2] : (w == 3) ? mk[3] : 0ull;
                const uint64_t hi = (w == 0) ? mk[1] : (w == 1) ? mk[2] : (w == 2) ? mk[3] : 0ull;
                win = (uint32_t)(sh ? ((lo >> sh) | (hi << (64 - sh))) : lo);
            }
            vbits = win >> (4 * g);
        }
        float p[16];
        float mx = -1e30f;
        if (SHARE && n0 <= -32) {   // keys every node sees
#pragma clang fp contract(off)      // the product is rounded before the maximum is taken off, as where it is tested
#pragma unroll
            for (int i = 0; i < 16; ++i) { p[i] = s[i] * a.scale; mx = fmaxf(mx, p[i]); }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const bool vis = (vbits >> (8 * (i >> 2) + (i & 3))) & 1u;   // key 8*(i/4) + 4*g + i%4 of the block
                p[i] = vis ? s[i] * a.scale : -1e30f;
                mx = fmaxf(mx, p[i]);
            }
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // Lazy rescale: the running reference m_run only has to be near the running maximum, not equal
        // to it -- exp(score - m_run) stays below e^8 as long as no row's maximum has grown by more than
        // 8 since the reference was set, which fp32 sums and bf16 probabilities hold without loss.  The
        // accumulators (64 registers, a read-multiply-write each) are rescaled only when some row of the
        // wavefront crosses that bound; after the first blocks of a long key range that is rare.
        const float m_cand = fmaxf(m_run, mx);
        if (__any(m_cand - m_run > 8.f)) {
            const float alpha = __expf(m_run - m_cand);
            l_run *= alpha;
            m_run = m_cand;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
        }
        float psum = 0.f;
        if (SHARE && n0 <= -32) {
            // What the test below leaves out counts for nothing here either: a score that is no number, and one of -1e29 or less while the
            // reference, which starts at -1e30, is that low too; against the next number above -1e29 its exponential is zero.
            const float m_ref = fmaxf(m_run, -0x1.431e0ep+96f);
#pragma unroll
            for (int i = 0; i < 16; ++i) { p[i] = fmaxf(__expf(p[i] - m_ref), 0.f); psum += p[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                p[i] = (p[i] > -1e29f) ? __expf(p[i] - m_run) : 0.f;
                psum += p[i];
            }
        }
        l_run += psum;
        uint4 pb[NQ], pbl[SPLIT ? NQ : 1];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if constexpr (SPLIT) pb[q] = Tr<EL>::pack_split(p + q * E, pbl[q]);   // what the probabilities lose to bf16 rounding goes through the matrix cores too
            else pb[q] = Tr<EL>::pack(p + q * E);
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                o[db] = Tr<EL>::mma(vt[db * NQ + q], pb[q], o[db]);
                if constexpr (SPLIT) o[db] = Tr<EL>::mma(vt[db * NQ + q], pbl[q], o[db]);
            }
    };
    // K of the next block is asked for when this block's has been multiplied, and arrives during the softmax and V's products; V of the next when
    // those are done, and arrives during K's.  No register more than with all of a block asked for at its start, which for 256 items of 72 blocks (7B,
    // 2298 keys), one workgroup a compute unit, was 33.5 us a layer, 30.7 this way.  (The last block asks for itself again: in range, not used.)
    int kb = kb_lo + wave;
    uint4 kt[NF], vt[DB * NQ];
    load_k(kt, kb < nkb ? kb : nkb - 1);
    load_v(vt, kb < nkb ? kb : nkb - 1);
    __builtin_amdgcn_sched_barrier(0);
    for (; kb < kb_hi; kb += 4) {
        const int kb_next = kb + 4 < kb_hi ? kb + 4 : kb;
        use_block(kt, vt, kb, kb_next);
        __builtin_amdgcn_sched_barrier(0);
        load_v(vt, kb_next);
        __builtin_amdgcn_sched_barrier(0);
    }
    l_run += __shfl_xor(l_run, 32);

    // ---- merge the four wavefronts: all park their accumulators in LDS, wavefront w combines 32-feature block w (blocks beyond D/32
    // have no wavefront).  With all blocks combined by wavefront 0 this, and the stores behind it, took four times as long.
    float* so = smem;                              // [DB][4 wavefronts][4 quads][64 lanes][4]
    float* sm = smem + 4 * DB * 64 * 16;           // [4][32] running max
    float* sl = sm + 4 * 32;                       // [4][32] running sum
    if constexpr (SHARE) __syncthreads();          // q lies there
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            ((float4*)so)[((db * 4 + wave) * 4 + q) * 64 + lane] = make_float4(o[db][4 * q], o[db][4 * q + 1], o[db][4 * q + 2], o[db][4 * q + 3]);
    if (g == 0) { sm[wave * 32 + tl] = m_run; sl[wave * 32 + tl] = l_run; }
    __syncthreads();
    int* ticket_lds = (int*)(sl + 4 * 32);
    float M = -1e30f, lsum = 0.f;
    float r[16];
    if (wave < DB) {
#pragma unroll
        for (int w = 0; w < 4; ++w) M = fmaxf(M, sm[w * 32 + tl]);
        float wgt[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) { wgt[w] = __expf(sm[w * 32 + tl] - M); lsum += wgt[w] * sl[w * 32 + tl]; }
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 v = ((const float4*)so)[((wave * 4 + w) * 4 + q) * 64 + lane];
                if (w == 0) { r[4 * q] = wgt[0] * v.x; r[4 * q + 1] = wgt[0] * v.y; r[4 * q + 2] = wgt[0] * v.z; r[4 * q + 3] = wgt[0] * v.w; }
                else { r[4 * q] += wgt[w] * v.x; r[4 * q + 1] += wgt[w] * v.y; r[4 * q + 2] += wgt[w] * v.z; r[4 * q + 3] += wgt[w] * v.w; }
            }
    }
    if (a.ks == 1) {
        if (wave < DB) {
            const float inv = (lsum > 0.f) ? 1.f / lsum : 0.f;
#pragma unroll
            for (int blk = 0; blk < 4; ++blk)
                store4_act<EL>(a.out, a.ld, qh * D + wave * 32 + 8 * blk + 4 * g, t, r[4 * blk] * inv, r[4 * blk + 1] * inv, r[4 * blk + 2] * inv,
                               r[4 * blk + 3] * inv);
        }
        return;
    }
    // ---- several workgroups share this item: partial triple out (agent-scope atomic stores,
    // acknowledged), ticket, and the last arriver combines all parts in part order
    constexpr int PF = FV_ATTN_PART_FLOATS(D);
    if (wave < DB) {
        float* pp = a.part + (size_t)(item * a.ks + part) * PF + lane;
#pragma unroll
        for (int i = 0; i < 16; ++i) __hip_atomic_store(pp + (wave * 16 + i) * 64, r[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (wave == 0 && g == 0) {
            __hip_atomic_store(pp + DB * 1024, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);         // lanes 0..31
            __hip_atomic_store(pp + DB * 1024 + 32, lsum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        handoff_release();
    }
    __syncthreads();   // every wavefront's stores are acknowledged
    if (tid == 0) *ticket_lds = __hip_atomic_fetch_add(&a.tickets[item], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    handoff_acquire();
    if (*ticket_lds != a.ks - 1) return;
    if (tid == 0) __hip_atomic_store(&a.tickets[item], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next use
    // wavefront w combines 32-feature block w (blocks beyond D/32 have no wavefront).  Everything it
    // needs from the up to eight parts is requested in one go, so the merge costs one memory round trip.
    const float* base = a.part + (size_t)item * a.ks * PF;
    for (int db = wave; db < DB; db += 4) {
        float mc[8], lc[8], v[8][16];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (c < a.ks) {   // the same in all lanes
                const float* cp = base + (size_t)c * PF;
                mc[c] = __hip_atomic_load(cp + DB * 1024 + tl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                lc[c] = __hip_atomic_load(cp + DB * 1024 + 32 + tl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int i = 0; i < 16; ++i) v[c][i] = __hip_atomic_load(cp + (db * 16 + i) * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                mc[c] = lc[c] = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) v[c][i] = 0.f;
            }
        }
        float Mx = -1e30f;
#pragma unroll
        for (int c = 0; c < 8; ++c) if (c < a.ks) Mx = fmaxf(Mx, mc[c]);
        float accv[16], ltot = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) accv[i] = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {   // part order
            const float wc = (c < a.ks) ? __expf(mc[c] - Mx) : 0.f;
            ltot += wc * lc[c];
#pragma unroll
            for (int i = 0; i < 16; ++i) accv[i] += wc * v[c][i];
        }
        const float inv = (ltot > 0.f) ? 1.f / ltot : 0.f;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk)
            store4_act<EL>(a.out, a.ld, qh * D + db * 32 + 8 * blk + 4 * g, t, accv[4 * blk] * inv, accv[4 * blk + 1] * inv,
                                accv[4 * blk + 2] * inv, accv[4 * blk + 3] * inv);
    }
}

// grid = items * ks
template <typename EL, int D, bool SHARE>
__global__ __launch_bounds__(256, SHARE ? 2 : 1) void k_attn(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) float smem[FV_ATTN_SMEM_FLOATS(D)];   // (SHARE: q lies where the accumulators are parked at the end)
    // Workgroups go to the 8 XCDs round-robin (workgroup b runs on XCD b % 8) and every XCD has its
    // own L2, so all node blocks and key parts of a query head -- and the query heads that share a
    // KV head -- are given to workgroups of one XCD: a head's K/V then comes from HBM once and is
    // re-read from that L2, instead of once per XCD that touches it.  (Only locality depends on the
    // dispatch order; any other order computes the same thing.)
    if (a.pieces > 1) {   // this piece's rows, and the keys of the pieces before it
        const int r0 = 256 * (int)blockIdx.y;
        a.L += r0;
        a.T = (a.T - r0 < 256) ? a.T - r0 : 256;
        a.TK = a.T;
        a.q += r0;
        a.q_lo += r0;
        a.out = (char*)a.out + (size_t)r0 * 16;
    }
    int item = blockIdx.x / a.ks, part = blockIdx.x % a.ks;
    if ((a.Hq & 7) == 0) {
        const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
        const int TB = a.Tp >> 5, per_head = TB * a.ks;
        const int head = x * (a.Hq >> 3) + j / per_head, w = j % per_head;
        item = head * TB + w / a.ks;
        part = w % a.ks;
    }
    attn_body<EL, D, SHARE>(a, item, part, smem);
}

#include "fv_attn_canon.hpp"

// ============================================================================ argmax
// Greedy choice per node: wavefront shuffle reduction on (value, index), lowest index on ties.
// A row that holds a NaN or an infinity has no greedy choice: its entry becomes -1, which the
// scan turns into an error for the whole step.
struct ArgmaxArgs {
    const float* logits;   // [Tp][Vpad]
    int32_t* am;           // [Tp]
    int V, Vpad;
};

__device__ __forceinline__ void argmax_combine(float& v, int& i, float ov, int oi) {
    if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
}

// The greedy choice of one row, in thread 0; -1 if it has none.  NT threads: a row of 32000 values took 256 threads four rounds of requests (13 us for a
// single row), 1024 take one.  A row that they hold at once is asked for its largest value first and for the first place that has it then: one
// maximum and one addition a value (of zeros, which a NaN or an infinity turns into a NaN), where value and place together took five instructions and two trips
// through LDS for each step of the reduction (us a step, device time: 7B width, four layers, 49 rows 562.7 -> 557.9; 250 rows 1019 -> 1014).
template <int NT>
__device__ __forceinline__ int argmax_row(const float* row, int V) {
    __shared__ float sv[NT / 64];
    __shared__ int si[NT / 64];
    __shared__ int sbad[NT / 64];
    const int tid = threadIdx.x;
    if (V <= 32 * NT) {
        float4 x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int v = (tid + k * NT) * 4;
            x[k] = (v < V) ? *(const float4*)(row + v) : make_float4(-FLT_MAX, -FLT_MAX, -FLT_MAX, -FLT_MAX);   // (a row is padded to a multiple of 32)
            if (v + 1 >= V) x[k].y = -FLT_MAX;
            if (v + 2 >= V) x[k].z = -FLT_MAX;
            if (v + 3 >= V) x[k].w = -FLT_MAX;
        }
        float bv = -FLT_MAX, zero = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            bv = fmaxf(fmaxf(bv, x[k].x), x[k].y);
            bv = fmaxf(fmaxf(bv, x[k].z), x[k].w);
            zero = fmaf(x[k].x, 0.f, zero); zero = fmaf(x[k].y, 0.f, zero);
            zero = fmaf(x[k].z, 0.f, zero); zero = fmaf(x[k].w, 0.f, zero);
        }
        const float wv = wave_max(bv);
        const bool wbad = __any(!(zero == 0.f));
        if ((tid & 63) == 0) { sv[tid >> 6] = wv; sbad[tid >> 6] = wbad ? 1 : 0; }
        if (tid == 0) si[0] = 0x7fffffff;
        __syncthreads();
        float best = sv[0];
        int any = sbad[0];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) { best = fmaxf(best, sv[w]); any |= sbad[w]; }
        if (bv == best) {   // -0 and +0 are equal here too
            int at = 0x7fffffff;
#pragma unroll
            for (int k = 7; k >= 0; --k) {
                const int v = (tid + k * NT) * 4;
                if (x[k].w == best && v + 3 < V) at = v + 3;
                if (x[k].z == best && v + 2 < V) at = v + 2;
                if (x[k].y == best && v + 1 < V) at = v + 1;
                if (x[k].x == best && v < V) at = v;
            }
            atomicMin(&si[0], at);
        }
        __syncthreads();
        return any ? -1 : si[0];
    }
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    bool bad = false;
    // eight 16-byte loads in flight per thread (the row is a latency chain otherwise: one load per
    // trip of a loop the compiler does not pipeline); indices past Vpad are not touched, values
    // between V and Vpad are skipped
    for (int v0 = tid * 4; v0 < V; v0 += 8 * NT * 4) {
        float4 x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int v = v0 + k * NT * 4;
            x[k] = (v < V) ? *(const float4*)(row + v) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int v = v0 + k * NT * 4;
            const float xs[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (v + c < V) {
                    // finite <=> |x| < inf; false for NaN too
                    bad = bad || !(__builtin_fabsf(xs[c]) < INFINITY);
                    argmax_combine(bv, bi, xs[c], v + c);
                }
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float ov = __shfl_xor(bv, off);
        const int oi = __shfl_xor(bi, off);
        argmax_combine(bv, bi, ov, oi);
    }
    const bool wbad = __any(bad);
    if ((tid & 63) == 0) { sv[tid >> 6] = bv; si[tid >> 6] = bi; sbad[tid >> 6] = wbad ? 1 : 0; }
    __syncthreads();
    int any = sbad[0];
    for (int w = 1; w < NT / 64; ++w) { argmax_combine(bv, bi, sv[w], si[w]); any |= sbad[w]; }   // thread 0's value starts as its own wavefront's
    return any ? -1 : bi;
}

// Whether this thread's share of a row holds a NaN or an infinity (the sum of zeros of argmax_row)
template <int NT>
__device__ __forceinline__ bool row_has_non_finite(const float* row, int V) {
    float zero = 0.f;
    for (int v0 = threadIdx.x * 4; v0 < V; v0 += 8 * NT * 4) {
        float4 x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int v = v0 + k * NT * 4;
            x[k] = (v < V) ? *(const float4*)(row + v) : make_float4(0.f, 0.f, 0.f, 0.f);
            if (v + 1 >= V) x[k].y = 0.f;
            if (v + 2 >= V) x[k].z = 0.f;
            if (v + 3 >= V) x[k].w = 0.f;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            zero = fmaf(x[k].x, 0.f, zero); zero = fmaf(x[k].y, 0.f, zero);
            zero = fmaf(x[k].z, 0.f, zero); zero = fmaf(x[k].w, 0.f, zero);
        }
    }
    return !(zero == 0.f);
}

template <int NT>
static __global__ __launch_bounds__(NT) void k_argmax(ArgmaxArgs a) {
    const int best = argmax_row<NT>(a.logits + (size_t)blockIdx.x * a.Vpad, a.V);
    if (threadIdx.x == 0) a.am[blockIdx.x] = best;
}

// ============================================================================ non-greedy acceptance
// Multi-step speculative sampling over the tree (the non-greedy setting of the paper's Appendix
// "Tree Structure"; verification in the SpecInfer manner, section "Custom-Designed Decoding Tree").
// At a node with w = exp((logits[node] - max) / temperature): the children are tried in index order;
// child c with token x is accepted iff u_accept[c] * q[x] * sum(w) <= w[x]; on rejection w becomes the
// positive part of w - sum(w) * q and the next child is tried against it.  q is row `node` of
// draft_probs, or a point mass on x if draft_probs is null (then rejection just strikes x from w).
// When no child is accepted the next token is the first v with cumsum(w)[v] > u_sample[node] * sum(w).
// All of it in fp64 (the decisions are thresholds on sums of 32000 terms; fp64 keeps both sides of a
// comparison with a CPU implementation within ~1e-13 of each other), in a fixed order, so the result
// is reproducible.
//
// What a node decides does not depend on how it was reached, so every node is decided at the same time,
// one workgroup each (k_sampled_nodes), and the path is read off afterwards (k_finish).  One
// workgroup that walked the path node by node took 390 us at 33 nodes of vocabulary 32000, as much as
// three layers: a dozen passes over the vocabulary one after the other, through one compute unit; this way
// it takes 52 us.  A node's
// own passes are still serial: one over its logits (32 fp64 exponentials per thread) and one per
// rejected child over w and q (384 KB through one compute unit's caches).  w is kept in memory: in registers it would
// take half the register file of a compute unit, and the compiler spilled it.
struct SampledArgs {
    const int32_t* tok_in;     // [3][cap]: tokens, parent, depth
    int cap, T;
    const float* logits;       // [Tp][Vpad]
    int V, Vpad;
    double inv_temperature;
    const float* draft_probs;  // [T][V] or null
    const double* u_accept;    // [T]
    const double* u_sample;    // [T]
    double* work;              // [T][Vpad] w of every node
    int32_t* outcome;          // [T] child taken (> node), or -1 - token drawn, or FV_SAMPLED_BAD
    int32_t* am;               // [T] greedy choices (written by k_sampled_resident)
};

#define FV_SAMPLED_THREADS 1024
// 16-byte loads of the caller's array only where they are aligned
__host__ __device__ __forceinline__ bool sampled_vectors(const float* draft_probs, int V) { return draft_probs && (V & 3) == 0 && ((uintptr_t)draft_probs & 15) == 0; }
#define FV_SAMPLED_BAD ((int32_t)0x80000000)   // the node's logits hold a NaN or an infinity

// One group of the draw: this thread's four tokens from v on, whose wavefront's share begins at `at`; incl: the wavefront's mass up to and with this
// thread's.  The token drawn, if it is here, goes into s_pick.
__device__ __forceinline__ void sampled_draw(int v, const double (&w)[4], double at, double incl, double target, int lane, int& last, int& s_pick) {
    const double end = at + incl, prev = __shfl_up(incl, 1);
    double cum = lane > 0 ? at + prev : at;
    int pick = 0x7fffffff, mass = -1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        cum += w[e];
        if (w[e] > 0.0) { mass = v + e; if (pick == 0x7fffffff && cum > target) pick = v + e; }
    }
    if (mass >= 0) last = mass;
    if (!(end > target)) pick = 0x7fffffff;
    else if (pick == 0x7fffffff && mass >= 0) pick = mass;   // rounding inside the four
    const unsigned long long m = __ballot(pick != 0x7fffffff);   // tokens ascend with the lane
    if (m && lane == __builtin_ctzll(m)) atomicMin(&s_pick, pick);
}
__device__ __forceinline__ double sampled_scan(const double (&w)[4], int lane) {   // prefix sum over the wavefront
    double incl = (w[0] + w[1]) + (w[2] + w[3]);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    return incl;
}

template <typename LAST>   // the thread's last token with any mass: asked for only where nothing was picked
__device__ __forceinline__ void sampled_finish(const SampledArgs& a, int node, LAST last_with_mass, int& s_pick, int& s_flag) {
    __syncthreads();
    if (s_pick == 0x7fffffff) {   // target at or beyond the total (u_sample ~ 1 and rounding): the last token that has any mass
        const int last = last_with_mass();
        if (last >= 0) atomicMax(&s_flag, last + 1);
        __syncthreads();
        if (threadIdx.x == 0) a.outcome[node] = s_flag > 0 ? -s_flag : FV_SAMPLED_BAD;
    } else if (threadIdx.x == 0) {
        a.outcome[node] = -1 - s_pick;
    }
}

static __global__ __launch_bounds__(FV_SAMPLED_THREADS) void k_sampled_nodes(SampledArgs a) {
    constexpr int NW = FV_SAMPLED_THREADS / 64, STRIDE = 4 * FV_SAMPLED_THREADS;   // a thread's tokens: four neighbours of every group of 4096
    __shared__ double s_sum[2][NW];
    __shared__ float s_max[NW];
    __shared__ unsigned long long s_kids[FV_MAX_TREE / 64];
    __shared__ int s_flag, s_pick;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int node = blockIdx.x, V = a.V;
    const int32_t* tok = a.tok_in;
    const int32_t* parent = a.tok_in + a.cap;
    const float* row = a.logits + (size_t)node * a.Vpad;      // rows of logits and of work are padded to 32 values
    double* work = a.work + (size_t)node * a.Vpad;
    const float* q = a.draft_probs ? a.draft_probs + (size_t)node * V : nullptr;
    const bool q16 = sampled_vectors(a.draft_probs, V);

    if (tid == 0) { s_flag = 0; s_pick = 0x7fffffff; }
    if (tid < FV_MAX_TREE) {   // the node's children as a bit mask
        const unsigned long long m = __ballot(tid > node && tid < a.T && parent[tid < a.T ? tid : 0] == node);
        if (lane == 0) s_kids[wave] = m;
    }
    // ---- largest logit
    float mx = -INFINITY;
    bool nf = false;
#pragma unroll 8
    for (int v = tid * 4; v < V; v += STRIDE) {
        const float4 r = *(const float4*)(row + v);
        const float xs[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (v + e < V) { nf = nf || !(__builtin_fabsf(xs[e]) < INFINITY); mx = fmaxf(mx, xs[e]); }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if (lane == 0) s_max[wave] = mx;
    __syncthreads();
    if (nf) s_flag = 1;
    __syncthreads();
    if (s_flag) {
        if (tid == 0) a.outcome[node] = FV_SAMPLED_BAD;
        return;
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) mx = fmaxf(mx, s_max[k]);
    const double zmax = (double)mx * a.inv_temperature;

    // sum of one value per thread, in a fixed order; every thread gets it.  Two areas in turn: one barrier per sum.
    int turn = 0;
    auto block_sum = [&](double v) -> double {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) s_sum[turn][wave] = v;
        __syncthreads();
        double r = 0.0;
#pragma unroll
        for (int k = 0; k < NW; ++k) r += s_sum[turn][k];
        turn ^= 1;
        return r;
    };
    auto store_w = [&](int v, const double (&w)[4]) {
        ((double2*)(work + v))[0] = make_double2(w[0], w[1]);
        ((double2*)(work + v))[1] = make_double2(w[2], w[3]);
    };
    auto load_w = [&](int v, double (&w)[4]) {
        const double2 lo = ((const double2*)(work + v))[0], hi = ((const double2*)(work + v))[1];
        w[0] = lo.x; w[1] = lo.y; w[2] = hi.x; w[3] = hi.y;
    };
    auto fill = [&]() -> double {   // w as it is before any rejection (zero beyond the vocabulary); its sum
        double ls = 0.0;
        for (int v = tid * 4; v < V; v += STRIDE) {
            const float4 r = *(const float4*)(row + v);
            const float xs[4] = {r.x, r.y, r.z, r.w};
            double w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w[e] = (v + e < V) ? exp((double)xs[e] * a.inv_temperature - zmax) : 0.0;
                ls += w[e];
            }
            store_w(v, w);
        }
        return block_sum(ls);
    };

    // ---- the children, in index order
    int taken = -1, wd = 0;
    unsigned long long kids = s_kids[0];
    double S = 0.0;
    for (;;) {
        if (!(S > 0.0)) S = fill();   // at first, and when nothing is left besides what was rejected (probability zero): the last p is kept
        while (!kids && ++wd < FV_MAX_TREE / 64) kids = s_kids[wd];
        if (!kids) break;
        const int c = wd * 64 + __builtin_ctzll(kids);
        kids &= kids - 1;
        const int t = tok[c];
        const double lhs = a.u_accept[c] * (q ? (double)q[t] : 1.0) * S, rhs = work[t];   // w[t] as the pass before left it: a barrier ago
        if (lhs <= rhs) { taken = c; break; }
        __syncthreads();              // everyone has read w[t] before it changes
        double ls = 0.0;
        if (q) {
#pragma unroll 4
            for (int v = tid * 4; v < V; v += STRIDE) {
                float qv[4] = {0.f, 0.f, 0.f, 0.f};
                if (q16) {
                    const float4 f = *(const float4*)(q + v);
                    qv[0] = f.x; qv[1] = f.y; qv[2] = f.z; qv[3] = f.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (v + e < V) qv[e] = q[v + e];
                }
                double w[4];
                load_w(v, w);
#pragma unroll
                for (int e = 0; e < 4; ++e) { w[e] = fmax(w[e] - S * (double)qv[e], 0.0); ls += w[e]; }
                store_w(v, w);
            }
        } else {
#pragma unroll 4
            for (int v = tid * 4; v < V; v += STRIDE) {
                double w[4];
                load_w(v, w);
#pragma unroll
                for (int e = 0; e < 4; ++e) { w[e] = (v + e == t) ? 0.0 : w[e]; ls += w[e]; }
                if (v == (t & ~3)) store_w(v, w);
            }
        }
        S = block_sum(ls);
    }
    if (taken >= 0) {
        if (tid == 0) a.outcome[node] = taken;
        return;
    }

    // ---- draw: the first v with cumsum(w)[v] > target, group after group in token order.  Every thread whose share ends above
    // the target proposes its first token with mass there, and the smallest token wins: a thread's share begins
    // exactly where its neighbour's ends, so no rounding can leave a gap between two.
    const double target = a.u_sample[node] * S;
    double base = 0.0;   // sum of the groups before
    int last = -1;       // this thread's last token with any mass
    for (int v0 = 0; v0 < V; v0 += STRIDE) {
        const int v = v0 + tid * 4;
        double w[4] = {0.0, 0.0, 0.0, 0.0};
        if (v < V) load_w(v, w);
        const double incl = sampled_scan(w, lane);
        if (lane == 63) s_sum[turn][wave] = incl;
        __syncthreads();
        double at = base;
        for (int k = 0; k < NW; ++k) { if (k == wave) at = base; base += s_sum[turn][k]; }
        turn ^= 1;
        sampled_draw(v, w, at, incl, target, lane, last, s_pick);
        if (base > target) break;   // the same in every thread
    }
    sampled_finish(a, node, [&]() { return last; }, s_pick, s_flag);
}

// Sums over a wavefront in every lane, by moves between registers instead of through LDS: the partners of the exchanges are those of shfl_xor with
// 32, 16 .. 1, or with 1, 2 .. 32 (where a pattern has other partners, these hold the same sums by then), so the sums are too, bit for bit.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, true), hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <int OFF>   // 16 or 32
__device__ __forceinline__ double swap_add(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t l = (uint32_t)b, h = (uint32_t)(b >> 32);
    const auto lo = OFF == 16 ? __builtin_amdgcn_permlane16_swap(l, l, false, false) : __builtin_amdgcn_permlane32_swap(l, l, false, false);
    const auto hi = OFF == 16 ? __builtin_amdgcn_permlane16_swap(h, h, false, false) : __builtin_amdgcn_permlane32_swap(h, h, false, false);
    return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) + __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}
__device__ __forceinline__ double wave_sum_from32(double v) {
    v = swap_add<16>(swap_add<32>(v));
    return dpp_add<0xB1>(dpp_add<0x4E>(dpp_add<0x124>(dpp_add<0x128>(v))));   // row_ror 8, 4; quad_perm 2,3,0,1 and 1,0,3,2
}
__device__ __forceinline__ double wave_sum_from1(double v) {
    v = dpp_add<0x140>(dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(v))));      // ...; row_half_mirror, row_mirror
    return swap_add<32>(swap_add<16>(v));
}

// The same decisions from the same sums for up to FV_SAMPLED_RESIDENT tokens, with w in registers and the greedy choice (k_argmax) found on the way:
// the logits are read once, w never leaves the compute unit, the node's row of the draft distribution comes to LDS while w is formed, and
// the draw adds up all groups before it looks into the one that the target lies in.  Half as many threads, each with the tokens and sums
// of two of the other kernel's (number tid and tid + 512): with one's share, 64 registers of 128, the compiler spilled it.  33 nodes of 32000
// tokens, argmax included: 61 -> 27 us (a node's two starts are most of it: the first look at its 128 KB, 5 us, and 64 fp64 exponentials a thread,
// 5 us; then 3 us a rejected child, and the draw).  With the row read again by every rejected child and the draw group by group: 61 -> 34.
// Q: there is a draft distribution, which sampled_vectors allows 16-byte loads of.  G: groups of 2048 tokens.  Those past the vocabulary cost as much as
// the others, so the host takes the fewest of 2, 4, 8 and 16 that hold it.  A call with 24 nodes (two layers of hidden 512; us without / with a draft
// distribution): 2000 tokens 143 / 131 in 16 groups, 124 / 122 in 2, 132 / 126 by k_argmax and k_sampled_nodes; 8000 tokens 145 / 141 in 16, 130 / 127 in 4,
// 141 / 139 by the two; 16000 tokens 147 / 139 in 16, 139 / 135 in 8, 155 / 147 by the two.  16 groups fill the registers: one value of eight bytes is in scratch.
#define FV_SAMPLED_GROUP (2 * FV_SAMPLED_THREADS)
#define FV_SAMPLED_RESIDENT (16 * FV_SAMPLED_GROUP)
template <bool Q, int G>
static __global__ __launch_bounds__(FV_SAMPLED_THREADS / 2) void k_sampled_resident(SampledArgs a) {
    constexpr int NT = FV_SAMPLED_THREADS / 2, NWH = NT / 64, NW = 2 * NWH;
    constexpr int STRIDE = FV_SAMPLED_GROUP;   // half of the other kernel's: even groups are the first thread's, odd ones the second's
    static_assert(STRIDE == 4 * NT && G % 2 == 0);
    __shared__ double s_sum[2][NW], s_w[2], s_tot[G][NWH];
    __shared__ float s_max[NWH];
    __shared__ int s_arg, s_bad[NWH];
    __shared__ unsigned long long s_kids[FV_MAX_TREE / 64];
    __shared__ int32_t s_tok[FV_MAX_TREE];
    __shared__ double s_u[FV_MAX_TREE];
    extern __shared__ uint4 sampled_q[];   // Q: G * FV_SAMPLED_GROUP floats, the node's row of the draft distribution
    __shared__ int s_flag, s_pick;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int node = blockIdx.x, V = a.V;
    const int32_t* parent = a.tok_in + a.cap;
    const float* q = Q ? a.draft_probs + (size_t)node * V : nullptr;
    // loads past a row's end give zeros: no branch in the loops over groups (the last vector of logits that has a token is inside Vpad)
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.logits + (size_t)node * a.Vpad), 0, ((V + 3) & ~3) * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t qrs = __builtin_amdgcn_make_buffer_rsrc((void*)q, 0, Q ? V * 4 : 0, 0x00020000);

    if (tid == 0) { s_flag = 0; s_pick = s_arg = 0x7fffffff; }
    if (tid < FV_MAX_TREE) {   // the node's children as a bit mask
        const unsigned long long m = __ballot(tid > node && tid < a.T && parent[tid < a.T ? tid : 0] == node);
        if (lane == 0) s_kids[wave] = m;
        s_tok[tid] = tid < a.T ? a.tok_in[tid] : 0;
        s_u[tid] = tid < a.T ? a.u_accept[tid] : 0.0;
    }
    auto here = [&]() {   // the thread's place in a group, in bytes (said to be new: sums with it are not kept in registers all the way through)
        unsigned o = tid * 16u;
        asm volatile("" : "+v"(o));
        return o;
    };
    int wd = -1, c = -1, t = 0, taken = -1;
    unsigned long long kids = 0;
    auto next_child = [&]() {   // in index order; c < 0: none left
        while (!kids && ++wd < FV_MAX_TREE / 64) kids = s_kids[wd];
        c = -1;
        if (!kids) return;
        c = wd * 64 + __builtin_ctzll(kids);
        kids &= kids - 1;
        t = s_tok[c];
    };
    double w[G][4];
    double S = 0.0;
    int turn = 0;
    for (bool first_time = true;; first_time = false) {   // again when nothing is left besides what was rejected (probability zero): the last p is kept
        float x[G][4];
        const unsigned o = here();
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const u32x4 r = __builtin_amdgcn_raw_buffer_load_b128(xrs, o + g * STRIDE * 4u, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[g][e] = __uint_as_float(r[e]);
        }
        // ---- largest logit
        int left = V - tid * 4;   // tokens from this thread's first on (said to be new, as above)
        asm volatile("" : "+v"(left));
        float own = -INFINITY, nf = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int e = 0; e < 4; ++e) nf = fmaf(x[g][e], 0.f, nf);   // no longer zero behind a NaN or an infinity
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[g][e] = g * STRIDE + e < left ? x[g][e] : -INFINITY;
                own = x[g][e] > own ? x[g][e] : own;
            }
            __builtin_amdgcn_sched_barrier(0);   // group by group, as they arrive
        }
        float mx = own;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        const bool wave_nf = __any(nf != 0.f);
        if (lane == 0) { s_max[wave] = mx; s_bad[wave] = wave_nf; }
        __syncthreads();
        bool bad = false;
#pragma unroll
        for (int k = 0; k < NWH; ++k) { mx = fmaxf(mx, s_max[k]); bad |= s_bad[k] != 0; }
        if (bad) {
            if (tid == 0) { a.am[node] = -1; a.outcome[node] = FV_SAMPLED_BAD; }
            return;
        }
        if (own == mx) {   // lowest token first, here and among the threads that have it
            int at = 0;
#pragma unroll
            for (int k = 4 * G - 1; k >= 0; --k) at = x[k >> 2][k & 3] == mx ? (k >> 2) * STRIDE + (k & 3) : at;
            atomicMin(&s_arg, at + tid * 4);
        }
        if (first_time) {
            next_child();
            if (Q && c >= 0) {   // the row is on its way while w is formed
                typedef __attribute__((address_space(3))) void* lptr;
#pragma unroll
                for (int g = 0; g < G; ++g)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(qrs, (lptr)(sampled_q + g * NT + wave * 64), 16, tid * 16 + g * STRIDE * 4, 0, 0, 0);
            }
        }

        // ---- w before any rejection (zero beyond the vocabulary).  ls[k]: the sum of what is thread tid + 512 k's in the other kernel
        const double zmax = (double)mx * a.inv_temperature;
        double ls[2] = {0.0, 0.0};
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w[g][e] = exp((double)x[g][e] * a.inv_temperature - zmax);
                ls[g & 1] += w[g][e];
            }
            if (g & 1) __builtin_amdgcn_sched_barrier(0);   // eight at a time
        }
        // ---- the children, in index order
        bool again = false;
        for (bool filled = true;; filled = false) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(w[g][e]));   // w stays where it is
            // the sum, in the other kernel's order, and the next child's w; every thread gets them.  Two areas in turn: one barrier.
#pragma unroll
            for (int k = 0; k < 2; ++k) ls[k] = wave_sum_from32(ls[k]);
            if (lane == 0) { s_sum[turn][wave] = ls[0]; s_sum[turn][NWH + wave] = ls[1]; }
            if (c >= 0 && ((t >> 2) & (NT - 1)) == tid) {
                const int at = t - tid * 4;
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (at == g * STRIDE + e) s_w[turn] = w[g][e];
            }
            if (Q && filled) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wavefront's share of the row is in LDS
            __syncthreads();
            S = 0.0;
#pragma unroll
            for (int k = 0; k < NW; ++k) S += s_sum[turn][k];
            const double w_t = s_w[turn];
            turn ^= 1;
            again = !(S > 0.0) && !filled;
            if (again || c < 0) break;
            if (s_u[c] * (Q ? (double)((const float*)sampled_q)[t] : 1.0) * S <= w_t) { taken = c; break; }
            const int struck = t - tid * 4;
            next_child();
            ls[0] = ls[1] = 0.0;
            if constexpr (Q) {
                int left = V - tid * 4;
                asm volatile("" : "+v"(left));
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float4 f = ((const float4*)sampled_q)[g * NT + tid];
                    const bool in = g * STRIDE < left;   // all four or none (sampled_vectors); past the row's end LDS holds anything
                    const float qv[4] = {in ? f.x : 0.f, in ? f.y : 0.f, in ? f.z : 0.f, in ? f.w : 0.f};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        w[g][e] = fmax(w[g][e] - S * (double)qv[e], 0.0);
                        ls[g & 1] += w[g][e];
                    }
                }
            } else {
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        w[g][e] = g * STRIDE + e == struck ? 0.0 : w[g][e];
                        ls[g & 1] += w[g][e];
                    }
            }
        }
        if (!again) break;
    }
    if (tid == 0) a.am[node] = s_arg;
    if (taken >= 0) {
        if (tid == 0) a.outcome[node] = taken;
        return;
    }

    // ---- draw, as in k_sampled_nodes, but all groups' sums first: only the group that the target lies in is looked into
    const double target = a.u_sample[node] * S;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const double total = wave_sum_from1((w[g][0] + w[g][1]) + (w[g][2] + w[g][3]));   // the last lane's of sampled_scan
        if (lane == 0) s_tot[g][wave] = total;
    }
    __syncthreads();
    double base = 0.0, at[2] = {0.0, 0.0};
    int g2 = 0;
    for (; g2 < G && g2 * STRIDE < V; g2 += 2) {
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (k % NWH == wave) at[k / NWH] = base;
            base += s_tot[g2 + k / NWH][k % NWH];
        }
        if (base > target) break;   // the same in every thread
    }
    int last = -1;
#pragma unroll
    for (int g = 0; g < G; g += 2)
        if (g == g2) {
#pragma unroll
            for (int k = 0; k < 2; ++k) sampled_draw((g + k) * STRIDE + tid * 4, w[g + k], at[k], sampled_scan(w[g + k], lane), target, lane, last, s_pick);
        }
    sampled_finish(a, node, [&]() {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) if (g < g2 + 2 && w[g][e] > 0.0) last = g * STRIDE + tid * 4 + e;
        return last;
    }, s_pick, s_flag);
}

// ============================================================================ end of a step
// The accepted path, and what is kept of it: one launch.  Every workgroup finds the path by itself (a few KB of node data and
// a microsecond; handing it on would be a launch, 5 us with its gap, and a step of two small layers is 100 us) and then does its
// share:
//   workgroup 0 writes the result record, straight into the host's memory (a copy behind the launch is 3 us and its gap);
//   T workgroups, one per possible path position, write a feature row: the LM head's input (final RMSNorm of the last layer's
//     output) of path node j, j = 0..accepted_len, fp32 [max_tree][h];
//   the others compact the cache, 256 / D slabs (layer, KV head) each: slot L + j <- slot L + path[j], j = 0..accepted_len.
//     Tree K/V were written at slots L + node index; path[j] >= j and ascends, so a slot that a row is read from is written for
//     that row at the earliest: rows may be read ahead of the writes of earlier ones.
// Greedy: match[i] = (i is the root) or tok[i] == argmax[parent[i]]; node i is accepted iff every node of its ancestor set
// matches; best = deepest accepted node, lowest index among equals; path = members of best's ancestor set in increasing index
// (= depth) order.  SAMPLED: from the root along the children the nodes took, to the token drawn at the end.
struct FinishArgs {
    const int32_t* tok_in;     // [3][cap]
    int cap, T;
    const uint64_t* mask;      // greedy
    const int32_t* am;         // [Tp]
    const int32_t* outcome;    // SAMPLED: [T], see SampledArgs
    const uint32_t* fault;
    FvResult* res;             // host memory
    // features
    const float* x;            // residual stream after the last layer, fp32 [h/4][Tp][4]
    const float* ssq;          // its per-strip sums of squares [h/32][Tp]
    const float* gain;         // final norm gain [h]
    float* feat;               // [max_tree][h]
    int h, Tp;
    float inv_h, eps;
    // compaction
    void* kcache;              // [slabs][S_pad*D]
    void* vcache;
    int slabs, L, S_pad;
};

// Features of row t, the b-th of the path, by NT threads; the first 256 add up the statistics
template <int NT>
__device__ __forceinline__ void finish_feature(const FinishArgs& a, int t, int b, float* red) {
    const int i = threadIdx.x;
    if (i < 256) {
        float s = 0.f;
        for (int k = i; k < a.h / 32; k += 256) s += a.ssq[(size_t)k * a.Tp + t];
        red[i] = s;
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (i < w) red[i] += red[i + w];
        __syncthreads();
    }
    const float rinv = rsqrtf(red[0] * a.inv_h + a.eps);
    for (int f0 = i; f0 < a.h; f0 += 8 * NT) {   // eight values read before the first is stored: one trip to memory for them, not one each
        float x[8], gn[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int f = f0 + k * NT < a.h ? f0 + k * NT : f0;
            x[k] = a.x[((size_t)(f >> 2) * a.Tp + t) * 4 + (f & 3)];
            gn[k] = a.gain[f];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (f0 + k * NT < a.h) a.feat[(size_t)b * a.h + f0 + k * NT] = x[k] * rinv * gn[k];
    }
}

// The end of a greedy step of one node, whose path is known: its greedy choice and the step's result, and beside it its features.  (Nothing moves in the cache.)
// Plain decoding pays for one launch here instead of two: one token of the 7B width, four layers 441.8 -> 432.6 us of device time, of hidden 512, two layers 84.5 -> 81.0.
// (Both workgroups read the logits, the second so that a step without a choice exports nothing: under the profiler 3.5 us a launch instead of 2.9 at 2000 tokens, 5.8
// instead of 4.3 at 32000; a call of hidden 512 91.7 us without, 91.0 with it, of the 7B width 466 and 467.  Its loads ahead of the statistics: 0.2 and 0.4 us less, not kept.)
template <int NT>
static __global__ __launch_bounds__(NT) void k_finish_one(ArgmaxArgs am, FinishArgs a) {
    __shared__ float red[256];
    if (blockIdx.x == 1) {   // a step without a choice leaves the features of the step before
        if (!__syncthreads_or(row_has_non_finite<NT>(am.logits, am.V))) finish_feature<NT>(a, 0, 0, red);
        return;
    }
    const int best = argmax_row<NT>(am.logits, am.V);
    if (threadIdx.x == 0) {
        am.am[0] = best;
        a.res->accepted_len = best < 0 ? FV_SCAN_NONFINITE : 0;
        a.res->next_token = best;
        a.res->best = 0;
        a.res->rows.fault = *a.fault;
        if (best >= 0) a.res->path[0] = 0;
        a.res->rows.argmax[0] = best;
        __threadfence_system();
    }
}

template <typename EL, int D, bool SAMPLED>
__global__ __launch_bounds__(256) void k_finish(FinishArgs a) {
    __shared__ unsigned long long mbits[4];
    __shared__ int best_key, any_bad, s_len, s_next, s_best;
    __shared__ int32_t s_path[FV_MAX_TREE], s_tok[FV_MAX_TREE], s_out[SAMPLED ? FV_MAX_TREE : 1];
    __shared__ float red[256];
    const int i = threadIdx.x;
    const int32_t* tok = a.tok_in;
    const int32_t* parent = a.tok_in + a.cap;
    const int32_t* depth = a.tok_in + 2 * a.cap;
    if (i < a.T) s_tok[i] = tok[i];
    if constexpr (!SAMPLED) {
        if (i < 4) mbits[i] = 0ull;
        if (i == 0) { best_key = -1; any_bad = 0; }
        __syncthreads();
        uint64_t mk[4] = {0, 0, 0, 0};
        if (i < a.T) {
            if (a.am[i] < 0) any_bad = 1;   // a row without a greedy choice (non-finite logits)
            for (int w = 0; w < 4; ++w) mk[w] = a.mask[i * 4 + w];
            const bool match = (i == 0) || (s_tok[i] == a.am[parent[i]]);
            if (match) atomicOr(&mbits[i >> 6], 1ull << (i & 63));
        }
        __syncthreads();
        if (i < a.T) {
            bool ok = true;
            for (int w = 0; w < 4; ++w) ok = ok && ((mk[w] & ~mbits[w]) == 0ull);
            if (ok) atomicMax(&best_key, depth[i] * 512 + (511 - i));
        }
        __syncthreads();
        const int best = 511 - (best_key & 511);
        const uint64_t* mb = a.mask + best * 4;
        if (i < a.T && ((mb[i >> 6] >> (i & 63)) & 1ull)) {
            int rank = 0;
            for (int w = 0; w < (i >> 6); ++w) rank += __popcll(mb[w]);
            rank += __popcll(mb[i >> 6] & ((1ull << (i & 63)) - 1ull));
            s_path[rank] = i;
        }
        if (i == 0) {   // no decision: FV_SCAN_NONFINITE tells the host, nothing is kept
            s_best = any_bad ? 0 : best;
            s_len = any_bad ? FV_SCAN_NONFINITE : depth[best];
            s_next = any_bad ? -1 : a.am[best];
        }
    } else {
        if (i < a.T) s_out[i] = a.outcome[i];
        __syncthreads();
        if (i == 0) {
            int cur = 0, len = 0, o = s_out[0];
            s_path[0] = 0;
            while (o > cur && o < a.T) {   // a child's index is above its parent's: the walk ends
                cur = o;
                s_path[++len] = cur;
                o = s_out[cur];
            }
            const bool bad = o == FV_SAMPLED_BAD || o >= 0;
            s_best = bad ? 0 : cur;
            s_len = bad ? FV_SCAN_NONFINITE : len;
            s_next = bad ? -1 : -1 - o;
        }
    }
    __syncthreads();
    const int len = s_len;
    int b = blockIdx.x;
    if (b == 0) {
        if (i == 0) { a.res->accepted_len = len; a.res->next_token = s_next; a.res->best = s_best; a.res->rows.fault = *a.fault; }
        if (i <= len) {
            a.res->path[i] = s_path[i];
            if (i >= 1) a.res->accepted_tokens[i - 1] = s_tok[s_path[i]];
        }
        if (i < a.T) a.res->rows.argmax[i] = a.am[i];
        __threadfence_system();
        return;
    }
    if (--b < a.T) {
        if (b <= len) finish_feature<256>(a, s_path[b], b, red);
        return;
    }
    const int slab = (b - a.T) * (256 / D) + i / D, e = i % D;
    if (slab >= a.slabs) return;
    char* ks = (char*)a.kcache + (size_t)slab * a.S_pad * D * Tr<EL>::ESZ;
    char* vs = (char*)a.vcache + (size_t)slab * a.S_pad * D * Tr<EL>::ESZ;
    typedef typename Tr<EL>::elem_t el_t;
    for (int j0 = 0; j0 <= len; j0 += 4) {   // four rows read before the first is written
        el_t k[4], v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int src = s_path[j0 + c <= len ? j0 + c : len];
            k[c] = ((const el_t*)ks)[kcache_index<EL, D>(a.L + src, e)];
            v[c] = ((const el_t*)vs)[vcache_index<EL, D>(a.L + src, e)];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = j0 + c;
            if (j > len || s_path[j] == j) continue;
            ((el_t*)ks)[kcache_index<EL, D>(a.L + j, e)] = k[c];
            ((el_t*)vs)[vcache_index<EL, D>(a.L + j, e)] = v[c];
        }
    }
}

// ============================================================================ helpers: weight tiling, KV read-back
struct TileArgs {
    const void* src0; const void* src1; const void* src2;
    uint4* out;
    int kind, n_strips_pad, NB, K, N;
    int Hq, Hkv, D, F;
};

template <typename EL>
__global__ __launch_bounds__(256) void k_tile(TileArgs a) {
    constexpr int E = Tr<EL>::E;
    const size_t total = (size_t)a.n_strips_pad * a.NB * FV_FRAGS * 64;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int lane = idx & 63;
    // output order [strip pair][half K batch][strip of the pair][4 frags][64 lanes]
    const size_t tile = idx >> 6;
    const int ff = (int)(tile & 3), r = (int)((tile >> 2) & 1);
    const size_t pj = tile >> 3;
    const int j = (int)(pj % ((size_t)2 * a.NB));
    const int strip = 2 * (int)(pj / ((size_t)2 * a.NB)) + r;
    const int frag = 4 * j + ff;
    const int m = lane & 31, g = lane >> 5;
    const int k0 = frag * 2 * E + g * E;
    const void* src = nullptr;
    long long row = -1;
    if (a.kind == TILE_NAT) {
        row = (long long)strip * 32 + m;
        src = a.src0;
        if (row >= a.N) row = -1;
    } else if (a.kind == TILE_QKV) {
        const int sph = a.D / 32, head = strip / sph, j = strip % sph;
        const int blk = m >> 3, within = m & 7;
        const int paired = (blk & 1) * (a.D / 2) + 16 * j + (blk >> 1) * 8 + within;
        if (head < a.Hq) { src = a.src0; row = (long long)head * a.D + paired; }
        else if (head < a.Hq + a.Hkv) { src = a.src1; row = (long long)(head - a.Hq) * a.D + paired; }
        else if (head < a.Hq + 2 * a.Hkv) { src = a.src2; row = (long long)(head - a.Hq - a.Hkv) * a.D + 32 * j + m; }
    } else {
        const int blk = m >> 3;
        const int f = 16 * strip + (blk >> 1) * 8 + (m & 7);
        if (f < a.F) { row = f; src = (blk & 1) ? a.src1 : a.src0; }
    }
    uint4 v = make_uint4(0, 0, 0, 0);
    if (row >= 0 && k0 < a.K)   // K is a multiple of E, so a vector is all inside or all outside
        v = *(const uint4*)((const char*)src + ((size_t)row * a.K + k0) * Tr<EL>::ESZ);
    a.out[idx] = v;
}

struct ReadKvArgs {
    const void* kcache; const void* vcache;   // this layer's slabs
    float* k_out; float* v_out;               // [n][Hkv][D]
    int slot0, n, Hkv, S_pad;
};
template <typename EL, int D>
__global__ void k_read_kv(ReadKvArgs a) {
    const int e = threadIdx.x, kh = blockIdx.y, j = blockIdx.x;
    if (j >= a.n) return;
    const char* ks = (const char*)a.kcache + (size_t)kh * a.S_pad * D * Tr<EL>::ESZ;
    const char* vs = (const char*)a.vcache + (size_t)kh * a.S_pad * D * Tr<EL>::ESZ;
    const size_t o = ((size_t)j * a.Hkv + kh) * D + e;
    a.k_out[o] = Tr<EL>::load(ks, kcache_index<EL, D>(a.slot0 + j, e));
    a.v_out[o] = Tr<EL>::load(vs, vcache_index<EL, D>(a.slot0 + j, e));
}
