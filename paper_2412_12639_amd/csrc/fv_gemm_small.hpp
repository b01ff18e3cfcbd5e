// Products of small matrices for up to 64 tokens: one 32-row strip a workgroup over its whole K range, no exchange across workgroups.
//
// What bounds them.  Such a launch is latency from end to end: arguments, one round of loads, a few matrix instructions, sums through LDS, the epilogue's loads
// and stores; and a wavefront alone on its SIMD issues an instruction every eight cycles, so the general kernel's bookkeeping (ranges, slices, request
// stream, parked tiles) was a third of it.  Here every wavefront asks for all it will multiply in one go.  Both forms add in the order of
// the direct kernel (fv_gemm_direct.hpp) for the same split, so they give its bits.
//
// k_gemm_small: matrices whose strips the direct kernel gives to one workgroup each (up to 8 K batches): three wavefronts take a third of the batches each.
// k_gemm_small_split: matrices of up to 16 batches that the direct kernel splits over many workgroups, one to three batches each, and whose sums it
// exchanges through memory.  One wavefront a batch does the same in LDS: batch sums, sums of those that one workgroup would have had,
// and these in ascending order, without their lowest mantissa bit from the second on, which the exchange uses as its mark.
// Device time of a step, two layers of hidden 512: one bf16 token 81 us before, 65 with the first form, 61 with both; 23 fp32 nodes 127 and 116, and 117 with a second
// form of two batches a wavefront for their 22 batches, which the general kernel keeps.
// Both sides of the lines, device us of a step, four layers and a head of 2000 tokens, 1 / 32 / 64 nodes, both forms against the general kernel alone: bf16, hidden 256
// and 688 behind it 92 / 105 / 114 against 128 / 140 / 170, 512 and 1376 102 / 115 / 145 against 141 / 154 / 189, 1024 (8 batches) and 2752 131 / 143 / 168 against
// 151 / 163 / 199; fp32, 256 and 688 143 / 158 / 214 against 192 / 205 / 278, 512 (8 batches) and 1376 181 / 194 / 261 against 200 / 214 / 294.  The split form alone, 1 / 32 nodes, with it
// against without: bf16, 512 and 1376 102 / 115 against 112 / 126, 512 and 2048 (16 batches) 109 / 122 against 119 / 130; fp32, 256 and 688 143 / 158 against 156 / 167, 1024
// (16 batches) and 1024 233 / 248 against 241 / 252.
#pragma once
// (included from fv_kernels.hpp after fv_gemm_direct.hpp)

#define FV_SMALL_NB 8          // K batches of the first form
#define FV_SMALL_SPLIT_NB 16   // of the second, 9 at least: a wavefront each

// Weights and activations of one K batch (8 fragments of one strip, 8 * TB tiles of activations), as the direct form's stage
template <typename EL, int TB>
struct SmallBatch {
    uint4 w[FV_FRAGS], x[FV_FRAGS * TB];
    __device__ __forceinline__ void load(const GemmArgs& a, int strip, int b, int lane) {
        constexpr int Tp = TB * 32;
        const uint4* wp = a.Wt + (((size_t)(strip >> 1) * (2 * a.NB) + 2 * b) * 2 + (strip & 1)) * (4 * 64) + lane;
        const uint4* xp = a.X + (size_t)b * (2 * FV_FRAGS * Tp) + (lane >> 5) * Tp + (lane & 31);
#pragma unroll
        for (int f = 0; f < FV_FRAGS; ++f)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) x[f * TB + tb] = xp[f * (2 * Tp) + tb * 32];
#pragma unroll
        for (int i = 0; i < FV_FRAGS; ++i) w[i] = wp[(i < 4 ? i : i + 4) * 64];
    }
    __device__ __forceinline__ void multiply(floatx16 (&acc)[TB]) const {
#pragma unroll
        for (int f = 0; f < FV_FRAGS; ++f)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) acc[tb] = Tr<EL>::mma(w[f], x[f * TB + tb], acc[tb]);
    }
};

template <typename EL, int TB, int D, int EPI>
__global__ __launch_bounds__(256, 1) void k_gemm_small(GemmArgs a) {
    constexpr int Tp = TB * 32;
    constexpr bool with_norm = EPI != EPI_RESID;
    __shared__ __attribute__((aligned(16))) float sums[FV_STREAMERS * TB * 1024];   // [wavefront][tile][4 quads][64 lanes][4]
    __shared__ __attribute__((aligned(16))) float red_lds[with_norm ? 16 * Tp : 4], rinv_lds[Tp];
    const int tid = threadIdx.x, lane = tid & 63, strip = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    request_args(a);

    // RMSNorm factors as in the direct form: 16 slices of the strips' sums, two rows of each at most (the host checks)
    constexpr int C4 = Tp / 4;
    const int col = tid % C4, sl = tid / C4;
    float4 sv[2];
    if constexpr (with_norm) {
        const __amdgpu_buffer_rsrc_t srs = __builtin_amdgcn_make_buffer_rsrc((void*)a.ssq_in, 0, a.n_ssq * (Tp * 4), 0x00020000);
        const unsigned at = sl < 16 ? (unsigned)(sl * C4 + col) * 16u : 0x80000000u;
#pragma unroll
        for (int k = 0; k < 2; ++k) sv[k] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(srs, at + (unsigned)(k * 16 * (Tp * 4)), 0, 0));
    }

    // this wavefront's third of the batches: up to three of them
    const int b0 = a.NB * wave / FV_STREAMERS, n = wave < FV_STREAMERS ? a.NB * (wave + 1) / FV_STREAMERS - b0 : 0;
    SmallBatch<EL, TB> m[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (i < n) m[i].load(a, strip, b0 + i, lane);
    // what the epilogue of this wavefront's tile reads besides
    EpiPre pre;
    bool have_pre = false;
    if (wave < TB) {
        if constexpr (EPI == EPI_RESID) { resid_preload(a, Tp, strip, wave, lane, pre); have_pre = true; }
        if constexpr (EPI == EPI_QKV) have_pre = rope_preload<D>(a, strip, wave, lane, pre);
    }
    if constexpr (with_norm) {
        const float4 s4 = make_float4(sv[0].x + sv[1].x, sv[0].y + sv[1].y, sv[0].z + sv[1].z, sv[0].w + sv[1].w);
        if (sl < 16) ((float4*)red_lds)[sl * C4 + col] = s4;
    }
    floatx16 acc[TB];
    zero_acc<TB>(acc);
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (i < n) m[i].multiply(acc);
    if (wave < FV_STREAMERS) {
        float4* my = (float4*)sums + (size_t)wave * TB * 256 + lane;
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) my[(t * 4 + q) * 64] = make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
    }
    __syncthreads();
    if (wave >= TB) return;
    if constexpr (with_norm) {   // wavefront t needs the factors of its own 32 columns: both halves of it work them out
        float tot = 0.f;
        const int c = wave * 32 + (lane & 31);
#pragma unroll
        for (int p = 0; p < 16; ++p) tot += red_lds[p * Tp + c];
        rinv_lds[c] = rsqrtf(tot * a.inv_h + a.eps);
        __builtin_amdgcn_wave_barrier();
    }
    float r[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float4 sum = ((const float4*)sums)[(wave * 4 + q) * 64 + lane];
#pragma unroll
        for (int w_ = 1; w_ < FV_STREAMERS; ++w_) {
            const float4 v = ((const float4*)sums)[((w_ * TB + wave) * 4 + q) * 64 + lane];
            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        r[4 * q] = sum.x; r[4 * q + 1] = sum.y; r[4 * q + 2] = sum.z; r[4 * q + 3] = sum.w;
    }
    gemm_epilogue<EL, D, EPI, true>(a, Tp, strip, wave, lane, r, rinv_lds, pre, have_pre);
}

// Up to 32 tokens, the residual products.  NB wavefronts, 8 at least.
template <typename EL, int D>
__global__ __launch_bounds__(1024) void k_gemm_small_split(GemmArgs a) {
    extern __shared__ __attribute__((aligned(16))) float smem_dyn[];   // [NB batches][4 quads][64 lanes][4]; the sum overwrites the first
    const int tid = threadIdx.x, lane = tid & 63, strip = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    request_args(a);
    EpiPre pre;
    if (wave == 0) resid_preload(a, 32, strip, 0, lane, pre);
    {
        SmallBatch<EL, 1> m;
        m.load(a, strip, wave, lane);
        floatx16 acc[1];
        zero_acc<1>(acc);
        m.multiply(acc);
        float4* my = (float4*)smem_dyn + (size_t)wave * 256 + lane;
#pragma unroll
        for (int q = 0; q < 4; ++q) my[q * 64] = make_float4(acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]);
    }
    // batches [e[c], e[c + 1]) are one workgroup's in the split
    int w = a.tab_cf[strip];
    __syncthreads();
    if (tid < 512) {   // two of the tile's values each
        const float2* const at = (const float2*)smem_dyn + tid;
        float2 r = make_float2(0.f, 0.f);
        for (int b = 0; b < a.NB; ++w) {
            const int e_ = split_unit(a, w + 1) - strip * a.NB, e = e_ < a.NB ? e_ : a.NB;
            float2 s = at[(size_t)b * 512];
            for (int k = b + 1; k < e; ++k) {
                const float2 v = at[(size_t)k * 512];
                s.x += v.x; s.y += v.y;
            }
            if (b == 0) r = s;
            else {
                r.x += __uint_as_float(__float_as_uint(s.x) & ~1u);
                r.y += __uint_as_float(__float_as_uint(s.y) & ~1u);
            }
            b = e;
        }
        *(float2*)at = r;   // this thread alone has read the place
    }
    __syncthreads();
    if (wave != 0) return;
    float r[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 v = ((const float4*)smem_dyn)[q * 64 + lane];
        r[4 * q] = v.x; r[4 * q + 1] = v.y; r[4 * q + 2] = v.z; r[4 * q + 3] = v.w;
    }
    gemm_epilogue<EL, D, EPI_RESID, true>(a, 32, strip, 0, lane, r, nullptr, pre, true);
}
