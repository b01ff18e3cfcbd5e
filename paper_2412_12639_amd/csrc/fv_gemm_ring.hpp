// GEMM for more than 64 rows, bf16: both operands go through a ring of LDS stages that the memory system fills by
// itself (global loads with an LDS destination), and the wavefronts do nothing but read fragments and multiply.
//
// What bounds it.  At 128 / 256 rows a matrix is read once and multiplied by 128 / 256 columns: about as long in HBM as
// on the matrix cores, so both have to run at once.  A wavefront takes two strips x half of the columns (2 + TB/2 KiB of LDS
// reads per TB matrix instructions) and nothing passes through registers.  A compute unit takes in about 14 KiB per memory latency, and a
// wavefront whose load is not taken yet stands still with it, matrix instructions included; so four wavefronts (one a SIMD) do nothing
// but fill the ring, five (256 rows) or eight (128 rows) stages ahead, and the four that multiply issue no load at all.  With the
// loads in the multiplying wavefronts, one at a time between matrix instructions, the two took as long as their sum: a stage of a
// prompt's products 0.52 us, now 0.36 to 0.41, where the matrix instructions alone take 0.34 (1.6 PFLOP/s over the chip).
// (Eight multiplying wavefronts that load for themselves: 1 %.)  A step's products read HBM besides, at its latency: 256 rows 0.55.
//
// Measured (7B width), loads among the matrix instructions -> this: a prompt of 2000 rows, gate/up 445 -> 340 us, QKV 240 -> 192, O and
// down 147 -> 117 on average, that is 1060, 1050 and 1070 TFLOP/s (library 900 to 1220); 256 rows QKV 47.6 -> 42.4, gate/up 67.9 -> 62.0, head 91 -> 83;
// 13B width, 128 rows, gate/up 75.9 -> 69.7, QKV 45 -> 42, head 78 -> 69.
//
// Tile: four strips x TB * 32 columns, four wavefronts as 2 x 2 and a filling one for each.  A stage is 32 columns of K: two weight
// fragments of every strip (1 KiB each, as tiled in memory) and four 16-byte vectors of every column.  One barrier per stage, in its
// middle: the second half of a stage multiplies while the first fragments of the next one are read, and the slot that
// everybody has left by then is filled again.
//
// WIDE = false: up to 256 rows, one block of columns; the (row group, K batch) space is cut into G ranges as for k_gemm,
// partial tiles are stored and k_gemm_fix, launched behind, reduces them.
// WIDE = true: more rows (a prompt): tiles over the whole K range, column tiles of 256.  One workgroup per compute unit takes several,
// the ring running on from one into the next: the next tile's first stages come while this one's sums go through the epilogue
// (gate/up, five to six tiles each, 350 -> 340 us).
#pragma once
// (included from fv_kernels.hpp after k_gemm_fix)

constexpr int ring_slots(int TB) { return TB == 4 ? 9 : 6; }
constexpr int ring_stage_bytes(int TB) { return FV_R * 2048 + TB * 32 * 64; }
constexpr size_t ring_smem(int TB) { return (size_t)ring_slots(TB) * ring_stage_bytes(TB) + (size_t)TB * 32 * 12 + 4096; }

template <int N> __device__ __forceinline__ void wait_vm() {   // all but the N youngest vector memory operations of this wavefront
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

#define FV_RING_THREADS 512   // wavefronts 0..3 multiply, 4..7 fill the ring

template <int TB, int D, int EPI, bool WIDE>
__device__ __forceinline__ void gemm_ring_body(const GemmArgs& a) {
    constexpr int NS = ring_slots(TB), SB = ring_stage_bytes(TB), AB = FV_R * 2048;
    constexpr int RS = 2, CB = TB / 2, TT = TB * 32;    // strips and column blocks of a wavefront, columns of the tile
    constexpr int LX = TT / 64, LPS = 2 + LX;           // loads per wavefront and stage: one strip's weights, one of four vectors of every column
    static_assert(LPS * (NS - 2) <= 63, "the outstanding-load counter");
    extern __shared__ __attribute__((aligned(16))) char ring[];
    float* const rinv_lds = (float*)(ring + NS * SB);
    float* const red_lds = rinv_lds + 3 * TT;           // [1024]
    const int tid = threadIdx.x, lane = tid & 63, tl = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
    const bool filler = __builtin_amdgcn_readfirstlane(tid >> 8) != 0;
    const int wr = wave >> 1, wc = wave & 1;
    request_args(a);
    const int NST = 4 * a.NB;                           // stages of a row group
    const int ld = WIDE ? a.ld : TT;                    // rows of the activation buffers
    int g0, k0, n;                                      // first group, its first stage, stages
    // WIDE: workgroups go to the XCDs round-robin; XCD x has the row groups x, x + 8, .., and tile i there is column tile i mod their
    // number of its group i / their number, so that the tiles in flight at a time share weights and these come from HBM once and then
    // from that XCD's L2.  A workgroup takes every t_step-th tile.
    const int tiles = WIDE ? ld / TT : 1, xcd = blockIdx.x & 7, t_step = gridDim.x >> 3;
    int ti = blockIdx.x >> 3;
    auto group_of = [&](int i) { return (i / tiles) * 8 + xcd; };
    auto column_of = [&](int i) { return (i % tiles) * TT; };
    if constexpr (WIDE) {
        g0 = group_of(ti);
        if (g0 >= a.NG) return;
        const int mine = (a.NG - 1 - xcd) / 8 * tiles + tiles;   // tiles of this XCD
        k0 = 0; n = ((mine - 1 - ti) / t_step + 1) * NST;
    } else {
        const int u0 = split_unit(a, blockIdx.x), u1 = split_unit(a, blockIdx.x + 1);   // computed, not looked up, as in k_gemm
        g0 = (int)((unsigned)u0 / a.div_NB); k0 = 4 * (u0 - g0 * a.NB); n = 4 * (u1 - u0);
    }

    // ---- fill: wavefront w brings strip w's weights and vector w of the activations, through buffer descriptors (bounds-checked;
    // the place in the matrix is a scalar, the lane's share a constant)
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.Wt, 0, (int)((unsigned)a.NG * FV_R * a.NB * 8192u), 0x00020000);
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.X, 0, (int)((unsigned)a.NB * 256u * (unsigned)ld), 0x00020000);
    int fg = g0, fk = k0, fn = 0, fslot = 0, fi = ti, ft0 = WIDE ? column_of(ti) : 0, fpar = 0;   // group, stage inside it, stages issued, slot; tile, its first column, its factors' place
    unsigned wo = 0, xo = 0;
    // A matrix of 32 MiB and more, all that the L2s hold, goes past the caches in a step (a row group's K batch is 32 KiB).  Smaller ones are better read plainly,
    // also where the layers together are more than the memory-side cache holds.  us a step of 100 / 250 rows, all plainly, all past the caches, by this rule:
    // hidden 1024, 8 layers 569 / 698, 599 / 730, 563 / 693; hidden 2048, 2 layers 231 / 298, 251 / 318, 236 / 294, 6 layers 600 / 787, 618 / 803, 588 / 777;
    // 7B width, 2 layers 434 / 568, 411 / 538, 406 / 534; 13B 518 / 684, 477 / 660, 474 / 659.  From 64 MiB on instead: two
    // layers of hidden 3072, or of 4096 with eight key heads, 3 to 6 % faster at 100 rows, the 7B width equal with two layers and 1 to 2 % slower with six; from 128 MiB on that 1 to 2 % slower with either.
    const bool once = !WIDE && (unsigned)a.NG * (unsigned)a.NB >= 1024u;
    auto place = [&]() {                                // of the stage to fill next
        const int strip = fg * FV_R + wave;             // tiled [strip pair][half K batch][2 strips][4 frags]: a stage of a strip is 2 KiB
        wo = ((((unsigned)(strip >> 1) * (2 * a.NB) + (fk >> 1)) * 2 + (strip & 1)) * 4 + (fk & 1) * 2) * 1024u;
        xo = ((unsigned)(fk * 4 + wave) * (unsigned)ld + (unsigned)ft0) * 16u;
    };
    auto load = [&](int i) {                            // load i of the stage (a constant after unrolling)
        typedef __attribute__((address_space(3))) void* lptr;
        char* const w = ring + fslot * SB + wave * 2048;
        char* const x = ring + fslot * SB + AB + wave * (TT * 16);
        switch (i) {
            case 0:                                     // both of the strip's fragments
                if (once) {
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lptr)w, 16, lane * 16, (int)wo, 0, FV_READ_ONCE);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lptr)w, 16, lane * 16, (int)wo, 1024, FV_READ_ONCE);
                } else {
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lptr)w, 16, lane * 16, (int)wo, 0, 0);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lptr)w, 16, lane * 16, (int)wo, 1024, 0);
                }
                break;
            case 1: break;
            case 2: __builtin_amdgcn_raw_ptr_buffer_load_lds(xrs, (lptr)x, 16, lane * 16, (int)xo, 0, 0); break;
            case 3: __builtin_amdgcn_raw_ptr_buffer_load_lds(xrs, (lptr)x, 16, lane * 16, (int)xo, 1024, 0); break;
            case 4: __builtin_amdgcn_raw_ptr_buffer_load_lds(xrs, (lptr)x, 16, lane * 16, (int)xo, 2048, 0); break;
            case 5: __builtin_amdgcn_raw_ptr_buffer_load_lds(xrs, (lptr)x, 16, lane * 16, (int)xo, 3072, 0); break;
        }
    };
    auto filled = [&]() {
        ++fn;
        if (++fk == NST) {
            fk = 0;
            if constexpr (WIDE) { fi += t_step; fg = group_of(fi); ft0 = column_of(fi); fpar = fpar == 2 ? 0 : fpar + 1; }
            else ++fg;
        }
        if (++fslot == NS) fslot = 0;
    };
    auto fill = [&]() {
        place();
        if constexpr (WIDE && EPI != EPI_RESID) {       // with a tile's first stage, its columns' RMSNorm factors: 64 from each wavefront (one load more in flight only makes a wait longer)
            typedef __attribute__((address_space(3))) void* lptr;
            if (fk == 0) {
                const __amdgpu_buffer_rsrc_t rrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.rinv_out, 0, ld * 4, 0x00020000);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rrs, (lptr)(rinv_lds + fpar * TT + wave * 64), 4, lane * 4, (ft0 + wave * 64) * 4, 0, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < LPS; ++j) load(j);
        filled();
    };
    // stage s has landed, as far as this wavefront fills it (behind the last stage to fill, everything is waited for)
    auto landed = [&](int s) { if (s + NS - 3 < n) wait_vm<LPS * (NS - 3)>(); else wait_vm<0>(); };

    if (filler) {
        for (int i = 0; i < NS - 1 && fn < n; ++i) fill();
        if constexpr (EPI != EPI_RESID && !WIDE) __syncthreads();   // (the others' statistics)
        landed(0);
        __builtin_amdgcn_s_barrier();
        for (int s = 0; s + 1 < n; ++s) {
            landed(s + 1);
            __builtin_amdgcn_s_barrier();   // everybody's part of stage s + 1 is there, and everybody has left stage s - 1
            if (fn < n) fill();
        }
        return;
    }

    // ---- RMSNorm factors of the columns
    if constexpr (EPI != EPI_RESID && !WIDE) {
        constexpr int C4 = TT / 4, SL = 256 / C4, NP = 128 / SL;   // the first 128 strips' sums are out before the rings' first loads
        const int col = tid % C4, sl = tid / C4;
        const float4* sp = (const float4*)a.ssq_in + col;
        float4 s4 = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 v[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) v[k] = (sl + k * SL < a.n_ssq) ? sp[(size_t)(sl + k * SL) * C4] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < NP; ++k) { s4.x += v[k].x; s4.y += v[k].y; s4.z += v[k].z; s4.w += v[k].w; }
        for (int i = sl + NP * SL; i < a.n_ssq; i += SL) {
            const float4 u = sp[(size_t)i * C4];
            s4.x += u.x; s4.y += u.y; s4.z += u.z; s4.w += u.w;
        }
        ((float4*)red_lds)[sl * C4 + col] = s4;
        __syncthreads();
        if (tid < TT) {
            float tot = 0.f;
#pragma unroll
            for (int p = 0; p < SL; ++p) tot += red_lds[p * TT + tid];
            const float rv = rsqrtf(tot * a.inv_h + a.eps);
            rinv_lds[tid] = rv;
            if (blockIdx.x == 0) a.rinv_out[tid] = rv;   // for k_gemm_fix
        }
    }

    struct Frags { u32x4 w[RS], x[CB]; };
    auto read = [&](Frags& d, int slot, int f, int i) {   // fragment i (a constant) of half f, in the order they are used: strip 0, the column blocks, strip 1
        const char* s = ring + slot * SB;
        if (i == 0 || i > CB) d.w[i == 0 ? 0 : 1] = *(const u32x4*)(s + ((wr * RS + (i == 0 ? 0 : 1)) * 2 + f) * 1024 + lane * 16);
        else d.x[i - 1] = *(const u32x4*)(s + AB + ((2 * f + g) * TT + (wc * CB + i - 1) * 32 + tl) * 16);
    };
    floatx16 acc[RS][CB];
    auto clear = [&]() {
#pragma unroll
        for (int r = 0; r < RS; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[r][c][i] = 0.f;
    };
    // Multiplies a half stage; between(i) runs behind matrix instruction i.  The next half's fragments are read there, one at a time: a
    // wavefront issues in order, and a burst of reads ahead of the matrix instructions leaves the matrix cores idle meanwhile.
    auto mul = [&](const Frags& d, auto&& between) {
#pragma unroll
        for (int r = 0; r < RS; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, d.w[r]), __builtin_bit_cast(bf16x8_t, d.x[c]), acc[r][c], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                between(r * CB + c);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    constexpr int NM = RS * CB, NR = RS + CB;   // matrix instructions and fragment reads of a half stage
    static_assert(NR <= NM, "one behind a matrix instruction");

    // ---- what happens to the sums of a segment: the epilogue if it covered the whole K range, else partial tiles for k_gemm_fix
    auto flush = [&](int gi, int t0, const float* rinv, bool whole, int seg) {
        if (whole) {
            // one tile after the other (all of what they read would be spilled)
            auto preload = [&](int i, EpiPre& d) -> bool {
                const int strip = gi * FV_R + wr * RS + i / CB, tb = t0 / 32 + wc * CB + i % CB;
                if (strip >= a.n_strips) return false;
                if constexpr (EPI == EPI_RESID) { resid_preload(a, ld, strip, tb, lane, d); return true; }
                if constexpr (EPI == EPI_QKV) return rope_preload<D>(a, strip, tb, lane, d);
                return false;
            };
            auto tile = [&](int i, const EpiPre& pre, bool have) {
                const int strip = gi * FV_R + wr * RS + i / CB, tb = t0 / 32 + wc * CB + i % CB;
                float v[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e] = acc[i / CB][i % CB][e];
                int ln = lane;
                if constexpr (!WIDE && EPI == EPI_QKV && D == 64) asm volatile("" : "+v"(ln));   // else all tiles' addresses are computed ahead of the first, and spilled: with 512 threads a wavefront has 256 registers
                if (strip < a.n_strips) gemm_epilogue<BF16, D, EPI>(a, ld, strip, tb, ln, v, rinv, pre, have);
            };
            if constexpr (WIDE) {   // what the next one reads is requested before this one's stores
                EpiPre pre[2];
                bool have[2] = {preload(0, pre[0]), false};
#pragma unroll
                for (int i = 0; i < RS * CB; ++i) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (i + 1 < RS * CB) have[(i + 1) & 1] = preload(i + 1, pre[(i + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    tile(i, pre[i & 1], have[i & 1]);
                }
            } else {                // rarely here: its own is enough
#pragma unroll
                for (int i = 0; i < RS * CB; ++i) {
                    __builtin_amdgcn_sched_barrier(0);
                    EpiPre pre;
                    const bool have = EPI == EPI_RESID && preload(i, pre);
                    __builtin_amdgcn_sched_barrier(0);
                    tile(i, pre, have);
                }
            }
        } else {
            const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc((void*)a.part, 0, (int)a.part_bytes, 0x00020000);
#pragma unroll
            for (int r = 0; r < RS; ++r)
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    const unsigned o = ((unsigned)((((int)blockIdx.x * a.segmax + seg) * FV_R + wr * RS + r) * TB + wc * CB + c) * 1024u + (unsigned)lane * 4u) * 4u;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        u32x4 v;
                        v.x = __float_as_uint(acc[r][c][4 * q]); v.y = __float_as_uint(acc[r][c][4 * q + 1]);
                        v.z = __float_as_uint(acc[r][c][4 * q + 2]); v.w = __float_as_uint(acc[r][c][4 * q + 3]);
                        __builtin_amdgcn_raw_buffer_store_b128(v, prs, o + q * 1024u, 0, 0);
                    }
                }
        }
    };

    clear();
    __builtin_amdgcn_s_waitcnt(0xC07F);   // the LDS stores above
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    Frags p, q;
#pragma unroll
    for (int i = 0; i < NR; ++i) read(p, 0, 0, i);
    int gi = g0, k = k0, seg = 0, seg_k0 = k0, slot = 0, par = 0;
    for (int s = 0; s < n; ++s) {
        mul(p, [&](int i) { if (i < NR) read(q, slot, 1, i); });
        if (++slot == NS) slot = 0;
        if (s + 1 < n) __builtin_amdgcn_s_barrier();   // as above: stage s + 1 is there
        __builtin_amdgcn_sched_barrier(0);
        // the reads behind the last stage are of no use; without a branch around them their wait count is known
        mul(q, [&](int i) {
            if (i < NR) read(p, slot, 0, i);
        });
        if (++k == NST || s + 1 == n) {
            if constexpr (WIDE) {
                const int t0 = column_of(ti);
                flush(gi, t0, rinv_lds + par * TT - t0, true, 0);
                ti += t_step; gi = group_of(ti); par = par == 2 ? 0 : par + 1;
            } else {
                flush(gi, 0, rinv_lds, seg_k0 == 0 && k == NST, seg);
                ++seg; ++gi; seg_k0 = 0;
            }
            k = 0;
            clear();
            __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): nothing but fragment reads is pending where the loop closes, so that their waits can count
        }
    }
}

template <int TB, int D, int EPI, bool WIDE>
__global__ __launch_bounds__(FV_RING_THREADS, 1) void k_gemm_ring(GemmArgs a) { gemm_ring_body<TB, D, EPI, WIDE>(a); }

// What only a drafter's long commit has over so many rows: products without a norm and an epilogue of their own (the LSTM's input multiplications), and the
// head that looks at all rows and keeps few.
template <int D, int EPI>
__global__ __launch_bounds__(FV_RING_THREADS, 1) void k_gemm_commit(GemmArgs a) { gemm_ring_body<8, D, EPI, true>(a); }
