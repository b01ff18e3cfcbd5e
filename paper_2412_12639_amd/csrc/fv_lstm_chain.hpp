// The recurrent half of one LSTM layer over a chain of rows, as one launch: the recurrent matrix stays on the chip
// (registers and LDS of all compute units) while the rows follow each other.
//
// What bounds it.  A chain is serial: row t needs the hidden state of row t - 1.  As separate launches (gather, weight
// multiplication, cell) every row streams the whole 4h x h matrix again: 134 MB and 33 us per row and layer at hidden
// 4096, of which 23 us are the stream.  That matrix is 512 KiB per compute unit, and a compute unit has 512 KiB of
// vector registers and 160 KiB of LDS: each wavefront keeps three quarters of its share in registers and one in LDS, the
// matrix is read once per launch, and a row costs what the exchange of the hidden state (0.8 us from the own publication until the others' values are here),
// the state's way through LDS and 64 matrix instructions per wavefront (0.7), and the way from their sums through the cell to the next publication (0.3) cost
// (time stamps in wavefront 0 of all 256 workgroups, which agree to 1 %).
// A wavefront that has its SIMD to itself issues an instruction every 8.4 cycles, a matrix instruction every 16, and LDS delivers a wavefront's 1 KiB
// in 8: what is on a row's path is counted in instructions.  (Taking the state's operands from lanes of the same row by moves across lanes instead
// of from LDS, eight moves an instruction: 0.3 us a row more.)  The look at the others' values takes half a microsecond and has to come when they are there, about
// 0.4 us behind the own publication: what a wavefront does in between (states and input rows) costs nothing, a look that comes 0.3 us earlier
// costs another look, 0.3 us a row.
// Measured at hidden 4096: 500 rows 954 us per layer (27 us to read the matrix, 1.85 us a row; with five instructions for every word of the
// state, a cell with branches and exchanges through LDS 1020, 1.99 a row) against 16500 as separate launches; 4 rows 33 against 130.
//
// Split: workgroup w owns hidden units 16w .. 16w+15 with their four gates (four 16-row blocks); its four wavefronts
// take a quarter of the K range each, so a wavefront needs only a quarter of the previous hidden state.  The sums of the
// four wavefronts meet in LDS (one of a step's two barriers; the other is in front of the looks), wavefront 0 applies the cell and publishes 16 new values.
//
// Exchange: the hidden state is published as bf16 (what the weight multiplication takes) in two buffers used in turn, by
// write-through stores, and read past the caches.  No flag or barrier across workgroups: |h| <= 1, so bit 14 of its bf16
// pattern (the top exponent bit) is always zero, and carries the phase of the buffer's use instead; every 4-byte word
// says itself whether it has arrived.  (A NaN, the only other value a cell can give, would use that bit: with it cleared a
// NaN's pattern lies strictly above that of 1.0, where no finite state lies, so the reader restores it.)  A buffer is overwritten
// for step s + 2 only by a workgroup that has all of step s + 1, hence after every workgroup has read step s.
//
// All workgroups must be on the chip at the same time.  They say so first: each adds one to a counter, loads its
// weights, and starts only when the counter shows that everybody has arrived.  If that takes too long (other streams
// hold compute units), one of them turns the counter's top bit on, which all of them read as "leave": the launch ends
// without having written anything but *aborted, and the host runs the pass again as separate launches.  A launch behind one that
// left (the other layer's, a later tree pass's) finds *aborted set and leaves without the wait: an attempt costs one time-out.
// After a start nothing but the workgroups' own progress is waited for.
#pragma once
#include "fv_device.hpp"
#include "fv_draft_kernels.hpp"

struct LstmChainArgs {
    const uint4* Wt;       // tiled recurrent matrix [4h][h]
    const uint4* zeros;    // at least 1 KiB of zeros
    const float* g_in;     // [Tp][4h] input multiplication of the pass's rows
    const float* bias;     // [4h]
    float* state;          // this layer's state rows [257][2][h]
    void* xnext;           // [h/8][Tp][8] next layer's input, or null
    uint16_t* xchg;        // [2][h], zero when the launch starts
    uint32_t* sync;        // arrival counter, zero when the launch starts
    uint32_t* aborted;     // counts the launches whose workgroups did not get on the chip together
    uint32_t* fault;       // set to 1 when a published value did not arrive
    int t0, r0, n;         // the chain: pass rows t0 .. t0+n-1, state rows r0 + t0 ..  (t0 is 0; without it the compiler's addresses cost 45 ns a row)
    const float* from;     // [2][h] the state the first one continues
    int Tp, h;
    unsigned expect;       // arrivals to wait for (the grid; one more in the test of the give-up path)
    unsigned arrive_looks; // looks at the counter before giving up
    unsigned spin_limit;   // looks at a published value that has not arrived
};

// K fragments (32 columns) per wavefront, rounded up to a built size, and how many of them stay in registers: all, or three of
// every four (hidden 4096: 96 of 128 registers quads; 128 KiB of LDS for the rest)
constexpr int lstm_chain_reg_frags(int nkf) { return nkf > 16 ? nkf / 4 * 3 : nkf; }
constexpr size_t lstm_chain_smem(int nkf) {
    return ((size_t)4 * (nkf - lstm_chain_reg_frags(nkf)) * 4 * 64 + (size_t)4 * nkf * 4) * 16 + 2 * 4 * 4 * 16 * 4 + 16;
}

// Sigmoid, or tanh, of a gate: both from e = e^-|a| (a = x or 2x) and one quotient, without a branch (the library's functions, of which every lane ran
// both, took two thirds of the cell's 0.63 us).  A wavefront that has its SIMD to itself issues an instruction every eight cycles, so what counts in the cell
// is how many there are.  The exponential is the Taylor polynomial behind a reduction by multiples of ln 2: the hardware's own, a unit in the last
// place off, gave tanh a larger error than the library's.  tanh's numerator 1 - e comes from the same polynomial without the cancellation, with what its
// rounding lost beside it (a series of its own below 0.5, as before: ten instructions and two branches more).  Largest error against 64 bits,
// absolute and relative, of every 61st value of 1e-6 .. 128 and all around the ends of saturation, reciprocal exact or a unit off
// (tests/test_lstm_gate.py; in brackets the library's, 1e-6 .. 100): sigmoid 0.44e-7 and 1.18e-7 (0.89e-7 and 1.47e-7), tanh 0.62e-7 and 1.20e-7
// (0.82e-7 and 1.46e-7; with the series 0.67e-7 and 1.33e-7).  |result| <= 1, which the exchange relies on.
__device__ __forceinline__ float lstm_gate(float x, bool th) {
    const float ax = fabsf(x), ax2 = th ? ax + ax : ax, a = ax2 > 104.f ? 104.f : ax2;   // e^-104 is zero in 32 bits; no number stays none
    const float n = rintf(a * -1.44269504f), y = fmaf(n, 1.90465421e-9f, fmaf(n, -0.693147182f, -a));   // -a = n ln 2 + y
    float t = 1.f / 5040.f;
    t = fmaf(t, y, 1.f / 720.f);
    t = fmaf(t, y, 1.f / 120.f);
    t = fmaf(t, y, 1.f / 24.f);
    t = fmaf(t, y, 1.f / 6.f);
    t = fmaf(t, y, 0.5f);
    const float s = ldexpf(1.f, (int)n), ys = y * s;
    const float e = fmaf(fmaf(t, y, 1.f), ys, s);                                          // s + ys (1 + t y)
    const float b = (1.f - s) - ys, c = t * y, m = fmaf(-c, ys, b), m_lo = fmaf(-c, ys, b - m);   // 1 - e
    const float d = 1.f + e, d_lo = e - (d - 1.f);
    const float num = th ? m : (x >= 0.f ? 1.f : e), num_lo = th ? m_lo : 0.f;
    const float r0 = __builtin_amdgcn_rcpf(d);
    float r = num * r0;
    r = fmaf(r0, fmaf(-d_lo, r, fmaf(-d, r, num)) + num_lo, r);
    return th ? copysignf(r, x) : r;
}

// acc += a (two of every four columns) * w, the weights in accumulation registers or in vector registers.  Written out, because the compiler's
// form copies weights that live in accumulation registers to others before each use (eight moves an instruction, as long as two of
// them).  It does not see that this is a matrix instruction, so the wait states are written here: two in front, for an operand that a vector
// instruction has just written (500 pairs and a tree at the 7B width 4958 us without, 4961 with), and chain_mma_done() between the last
// of a row of them and the first use of acc.  That the compiler leaves acc alone in between is checked on the built code (tests/test_kernel_code.py).
typedef float chain_f4 __attribute__((ext_vector_type(4)));
typedef unsigned int chain_u4 __attribute__((ext_vector_type(4)));
typedef unsigned int chain_u8 __attribute__((ext_vector_type(8)));
template <bool ACC_REGS>
__device__ __forceinline__ void chain_mma(chain_f4& acc, const chain_u4& a, const chain_u8& w, int pick) {
    if constexpr (ACC_REGS) asm volatile("s_nop 1\n\tv_smfmac_f32_16x16x64_bf16 %0, %1, %2, %3" : "+v"(acc) : "v"(a), "a"(w), "v"(pick));
    else asm volatile("s_nop 1\n\tv_smfmac_f32_16x16x64_bf16 %0, %1, %2, %3" : "+v"(acc) : "v"(a), "v"(w), "v"(pick));
}
__device__ __forceinline__ void chain_mma_done(chain_f4 (&acc)[4]) {
    asm volatile("s_nop 15\n\ts_nop 3" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));
}

// The recurrent matrix, read once a launch: past the caches where it is as large as the L2s and more (33 and 134 MB).
template <int NKF> __device__ __forceinline__ uint4 ld_matrix(const uint4* p) { return NKF >= 16 ? ld_once(p) : *p; }

template <int NKF>
static __global__ __launch_bounds__(256, 1) void k_lstm_chain(LstmChainArgs a) {
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
    typedef unsigned int u32x8_t __attribute__((ext_vector_type(8)));
    typedef short short2_t __attribute__((ext_vector_type(2)));
    constexpr int NM = NKF / 2, RM = lstm_chain_reg_frags(NKF) / 2, LM = NM - RM;   // 64-column instructions per gate; with their weights in registers, in LDS
    constexpr int GM = NM < 4 ? NM : 4;
    constexpr int PIN = RM * 4 < 30 ? 0 : 30;   // weights in accumulation registers
    static_assert(NM % GM == 0 && (LM == 0 || LM == NM / 4), "whole groups");
    constexpr int NV = (4 * NKF + 63) / 64;        // 16-byte pieces of the hidden state per lane
    constexpr int SC1 = 16;
    constexpr unsigned LEAVE = 0x80000000u, TAG = 0x40004000u;
    extern __shared__ uint4 lds_chain[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int u = lane & 15, q = lane >> 4;
    const int wg = blockIdx.x, h = a.h;
    const int kf_real = h >> 7, quarter = h >> 2;
    uint4* const wl = lds_chain + (size_t)wave * LM * 8 * 64 + lane;                       // [LM][4 gates][2 halves][64 lanes] of this wavefront
    uint4* const hs = lds_chain + (size_t)4 * LM * 8 * 64 + (size_t)wave * NKF * 4;        // its quarter of the hidden state
    float* const part = (float*)(lds_chain + (size_t)4 * LM * 8 * 64 + (size_t)4 * NKF * 4);   // [2][4 wavefronts][4 gates][16]
    unsigned* const go = (unsigned*)(part + 2 * 4 * 4 * 16);

    if (tid == 0) __hip_atomic_fetch_add(a.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // weights: row block g = gate g, rows g*h + 16*wg ..; the matrix is tiled for 32-row strips and 16-column fragments, of
    // which a 16x16x32 operand takes half the rows of two neighbours.  Columns past h (sizes between the built ones) are zero.
    const int n_half = h >> 6;   // half K batches
    auto w_addr = [&](int g, int kf) {
        const int strip = g * (h >> 5) + (wg >> 1);
        const int F = wave * (h >> 6) + 2 * kf + (q >> 1);
        const uint4* p = a.Wt + ((((size_t)(strip >> 1) * n_half + (F >> 2)) * 2 + (strip & 1)) * 4 + (F & 3)) * 64 + (wg & 1) * 16 + u + 32 * (q & 1);
        return kf < kf_real ? p : a.zeros + lane;
    };
    u32x8_t w[RM][4];   // in K order; with some of them in LDS every fourth is there
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int m = LM > 0 ? i / 3 * 4 + i % 3 : i;
            const uint4 lo = ld_matrix<NKF>(w_addr(g, 2 * m)), hi = ld_matrix<NKF>(w_addr(g, 2 * m + 1));
            w[i][g] = u32x8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        }
    // The matrix instructions take their operand from the accumulation registers as well, but the compiler, left alone, parks
    // values there and copies them back before each use; said once that a value lives there, it uses it in place.
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (i * 4 + g < PIN) asm volatile("" : "+a"(w[i][g]));
    for (int i = 0; i < LM; ++i) {
        uint4 v[4][2];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 2; ++e) v[g][e] = ld_matrix<NKF>(w_addr(g, 2 * (4 * i + 3) + e));
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 2; ++e) wl[((i * 4 + g) * 2 + e) * 64] = v[g][e];
    }

    // The hidden state as the sparse operand.  A matrix instruction has sixteen columns for it and a chain one row, but the instruction for
    // matrices with two values in every four takes twice the K range in the same time; so even rows of the operand hold values 0 and 1 of
    // every four, odd rows values 2 and 3, and the result is the sum of an even and an odd row.  16 columns of K: 16 bytes for the even
    // rows, 16 for the odd ones.
    auto put_state = [&](int vec, uint4 v) {   // 8 values
        uint2* const p = (uint2*)hs + (vec >> 1) * 4 + (vec & 1);
        p[0] = make_uint2(v.x, v.z);
        p[2] = make_uint2(v.y, v.w);
    };
    const int pick = (u & 1) ? (int)0xEEEEEEEE : 0x44444444;   // which two of every four this lane's row has
    // the state the chain continues
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int vec = lane + 64 * j;
        if (vec < 4 * NKF) {
            float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (vec < 4 * kf_real) {
                const float4* sp = (const float4*)(a.from + wave * quarter + vec * 8);
                const float4 x0 = sp[0], x1 = sp[1];
                f[0] = x0.x; f[1] = x0.y; f[2] = x0.z; f[3] = x0.w; f[4] = x1.x; f[5] = x1.y; f[6] = x1.z; f[7] = x1.w;
            }
            put_state(vec, Tr<BF16>::pack(f));
        }
    }
    // wavefront 0: lane (q, u) owns gate q of unit u; every lane of a unit keeps the same cell state
    const size_t unit = (size_t)16 * wg + u;
    const float bias = a.bias[(size_t)q * h + unit];
    float c = a.from[h + unit];

    if (tid == 0) {
        // set here, *aborted is an earlier launch's, or this one's after its counter said "leave": nobody can start then
        const unsigned gone = __hip_atomic_load(a.aborted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned seen = 0;
        for (unsigned looks = 0;; ++looks) {
            seen = __hip_atomic_load(a.sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (gone) seen |= LEAVE;
            if ((seen & LEAVE) || seen == a.expect) break;
            if (looks >= a.arrive_looks) {   // "everybody is here" and "leave" exclude each other: one word decides
                unsigned old = seen;
                if (__hip_atomic_compare_exchange_strong(a.sync, &old, seen | LEAVE, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    seen |= LEAVE;
                    __hip_atomic_fetch_add(a.aborted, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // the one workgroup that decides it
                    break;
                }
                continue;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        *go = (seen & LEAVE) ? 0u : 1u;
    }
    __syncthreads();
    if (*go == 0u) return;

    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.xchg, 0, 4 * h, 0x00020000);
    const float* gin_p = a.g_in + (size_t)a.t0 * 4 * h + (size_t)q * h + unit;
    float gin = *gin_p;
    unsigned limit = a.spin_limit;
    // What a step needs besides its operands is ready before the barrier that it starts with
    int vec_of[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) vec_of[j] = ((lane + 64 * j < 4 * kf_real) ? lane + 64 * j : 4 * kf_real - 1) * 16 + wave * quarter * 2;
    const bool packs = q == 0 && (u & 1) == 0;                       // lanes that publish two units
    const unsigned pub = packs ? (unsigned)unit * 2u : 0x40000000u;  // elsewhere behind the end of the area: not stored
    for (int s = 0; s < a.n; ++s) {
        const float gin_now = gin + bias;
        if (s + 1 < a.n) gin_p += (size_t)4 * h;   // (the last step asks for its own again)
        gin = *gin_p;
        floatx4 acc[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
        u32x8_t wb[4];
        auto fetch_w = [&](int gr) {
            if constexpr (LM > 0) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const uint4 lo = wl[((gr * 4 + g) * 2) * 64], hi = wl[((gr * 4 + g) * 2 + 1) * 64];
                    wb[g] = u32x8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                }
            }
        };
        fetch_w(0);    // the first group's, while the state is waited for
        __builtin_amdgcn_sched_barrier(0);
        if (s > 0) {   // this wavefront's quarter of the state of step s - 1
            // Nobody looks for the others' values before this workgroup's own are out: the looks of three wavefronts that have nothing
            // else to do (8 KiB a workgroup and look, past the caches) held up everybody's stores (a row 2.57 -> 1.90 us).
            __builtin_amdgcn_s_barrier();
            const bool tagged = !(((s - 1) >> 1) & 1);
            const unsigned from = (unsigned)((s - 1) & 1) * 2u * (unsigned)h;
            u32x4_t v[NV];
            for (unsigned looks = 0;; ++looks) {
                asm volatile("" ::: "memory");   // a look is a look: the loads stay in the loop
#pragma unroll
                for (int j = 0; j < NV; ++j) v[j] = __builtin_amdgcn_raw_buffer_load_b128(xrs, vec_of[j] + from, 0, SC1);
                unsigned all = ~0u, any = 0u;
                if (tagged) {
#pragma unroll
                    for (int j = 0; j < NV; ++j) all = all & v[j].x & v[j].y & v[j].z & v[j].w;
                    any = ~all;
                } else {
#pragma unroll
                    for (int j = 0; j < NV; ++j) any = any | v[j].x | v[j].y | v[j].z | v[j].w;
                }
                if (__all((any & TAG) == 0u)) break;
                if (looks >= limit) {
                    limit = 0;   // the results are lost: the rest is not waited for either
                    if (lane == 0) __hip_atomic_store(a.fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
            }
            // What lies above 1.0 without its top exponent bit was a NaN (published as a positive one, so a maximum of signed halves finds it).
            short2_t top = short2_t{0, 0};
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int c_ = 0; c_ < 4; ++c_) {
                    v[j][c_] &= ~TAG;
                    top = __builtin_elementwise_max(top, __builtin_bit_cast(short2_t, (unsigned)v[j][c_]));
                }
            if (__any(top.x > 0x3F80 || top.y > 0x3F80)) {
#pragma unroll
                for (int j = 0; j < NV; ++j)
#pragma unroll
                    for (int c_ = 0; c_ < 4; ++c_) v[j][c_] |= (((v[j][c_] & 0x3fff3fffu) + 0x007f007fu) & TAG);
            }
#pragma unroll
            for (int j = 0; j < NV; ++j)   // (pieces past h repeat one in front of it: their weights are zero)
                if (64 * (j + 1) <= 4 * NKF || lane + 64 * j < 4 * NKF) put_state(lane + 64 * j, make_uint4(v[j].x, v[j].y, v[j].z, v[j].w));
        }
        __builtin_amdgcn_wave_barrier();   // hs belongs to this wavefront: LDS accesses of one wavefront stay in order
        asm volatile("s_nop 1" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));
        // groups of GM instructions a gate; the state of a group is read from LDS while the group before it multiplies, the weights of its
        // last instructions while its first ones do
        u32x4_t b[2][GM];
        auto fetch = [&](int gr, u32x4_t (&bd)[GM]) {
#pragma unroll
            for (int j = 0; j < GM; ++j) bd[j] = *(const u32x4_t*)&hs[((gr * GM + j) * 4 + q) * 2 + (u & 1)];
        };
        fetch(0, b[0]);
#pragma unroll
        for (int gr = 0; gr < NM / GM; ++gr) {
            if (gr > 0) fetch_w(gr);
            if (gr + 1 < NM / GM) fetch(gr + 1, b[(gr + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < GM; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if (LM > 0 && j == 3) { chain_mma<false>(acc[g], b[gr & 1][j], wb[g], pick); continue; }
                    const int i = LM > 0 ? (gr * 3 + j) % RM : gr * GM + j;
                    if (i * 4 + g < PIN) chain_mma<true>(acc[g], b[gr & 1][j], w[i][g], pick);
                    else chain_mma<false>(acc[g], b[gr & 1][j], w[i][g], pick);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_wave_barrier();
        chain_mma_done(acc);
        // every lane has an even and an odd row of each gate, for unit u: lane (q, u) hands on gate q
        float* const ps = part + (s & 1) * (4 * 4 * 16);   // [64 lanes][4 wavefronts]
        {
            const float even = q < 2 ? (q == 0 ? acc[0][0] : acc[1][0]) : (q == 2 ? acc[2][0] : acc[3][0]);
            const float odd = q < 2 ? (q == 0 ? acc[0][1] : acc[1][1]) : (q == 2 ? acc[2][1] : acc[3][1]);
            ps[lane * 4 + wave] = even + odd;
        }
        __syncthreads();   // part[s & 1] is next written after the barrier of step s + 1, which wavefront 0 reaches when it has read it
        if (wave == 0) {
            const float4 sums = ((const float4*)ps)[lane];
            const float pre = (((sums.x + sums.y) + sums.z) + sums.w) + gin_now;
            const float act = lstm_gate(pre, q == 2);
            // rows of lanes 0 .. 3 hold the four gates: every lane gets all of them by exchanging halves, then rows (through LDS it was four trips)
            const auto half = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, act), __builtin_bit_cast(unsigned, act), false, false);
            const auto in_f = __builtin_amdgcn_permlane16_swap(half[0], half[0], false, false), cell_o = __builtin_amdgcn_permlane16_swap(half[1], half[1], false, false);
            const float gi = __builtin_bit_cast(float, (unsigned)in_f[0]), gf = __builtin_bit_cast(float, (unsigned)in_f[1]);
            const float gg = __builtin_bit_cast(float, (unsigned)cell_o[0]), go_ = __builtin_bit_cast(float, (unsigned)cell_o[1]);
            c = gf * c + gi * gg;
            float hn = go_ * lstm_gate(c, true);
            hn = hn == hn ? hn : __builtin_nanf("");   // a positive one
            const float other = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, hn), 0xB1, 0xF, 0xF, false));   // the neighbour's
            const unsigned pair = pack_bf16x2(hn, other);   // even lanes: units u, u + 1
            __builtin_amdgcn_raw_buffer_store_b32((pair & ~TAG) | (((s >> 1) & 1) ? 0u : TAG), xrs, pub + (unsigned)(s & 1) * 2u * (unsigned)h, 0, SC1);
            const int t = a.t0 + s;
            if (q < 2) a.state[((size_t)(a.r0 + t) * 2 + q) * h + unit] = q == 0 ? hn : c;
            if (a.xnext && packs) *(unsigned*)((char*)a.xnext + ((unit >> 3) * a.Tp + t) * 16 + (unit & 7) * 2) = pair;
        }
    }
}

// The same for the levels of a tree pass: up to 16 rows a level, which are the 16 columns of the matrix instruction (a chain uses
// one of them).  At hidden 4096 a launch takes 31 us for one level, of which 25 read the matrix, and 5.5 for another (separate launches: gather 5, product
// 23 to 31, cell 5 us and gaps a level).  Differences to
// the chain: a level's rows continue rows anywhere in the level before, so a lane reads its column's predecessor; the first
// level's predecessors of both layers are gathered at the start of the pass, and layer 1 leaves what the decoder block takes in itself (a launch
// each of 5 us before; 2 us of layer 1's launch now); the operand goes from the exchange area straight to registers, a few
// fragments at a time; all four wavefronts apply the cell.
struct LstmLevelArgs {
    LstmChainArgs c;               // n, t0, from are not used; xchg: [2][h / 8][16][8]
    DraftTables tab;
    const uint4* xprev;            // [h / 8][32][8] bf16 predecessors' states of the first level
    float* x; void* xb; const float* gain; float* ssq;   // layer 1 (else null): residual stream, x * gain, and its sums of squares, zero when the launch starts, as k_lstm_out leaves them
    int l0, n_lvl;                 // first entry in lvl_rows; levels
    int rows[FV_DRAFT_KMAX];       // rows of each level, 1..16
};

constexpr size_t lstm_level_smem(int nkf) { return (size_t)4 * (nkf - lstm_chain_reg_frags(nkf)) * 4 * 64 * 16 + 4 * 4 * 16 * 16 * 4 + 16; }

template <int NKF>
static __global__ __launch_bounds__(256, 1) void k_lstm_levels(LstmLevelArgs la) {
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
    constexpr int RKF = lstm_chain_reg_frags(NKF), LKF = NKF - RKF;
    constexpr int GF = NKF < 4 ? NKF : 4;
    constexpr int SC1 = 16;
    constexpr unsigned LEAVE = 0x80000000u, TAG = 0x40004000u;
    extern __shared__ uint4 lds_chain[];
    const LstmChainArgs& a = la.c;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int u = lane & 15, q = lane >> 4;
    const int wg = blockIdx.x, h = a.h;
    const int kf_real = h >> 7;
    uint4* const wl = lds_chain + (size_t)wave * LKF * 4 * 64 + lane;
    float* const part = (float*)(lds_chain + (size_t)4 * LKF * 4 * 64);   // [4 wavefronts][4 gates][16 columns][16 units]
    unsigned* const go = (unsigned*)(part + 4 * 4 * 16 * 16);

    if (tid == 0) __hip_atomic_fetch_add(a.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int n_half = h >> 6;
    auto w_addr = [&](int g, int kf) {   // as in k_lstm_chain
        const int strip = g * (h >> 5) + (wg >> 1);
        const int F = wave * (h >> 6) + 2 * kf + (q >> 1);
        const uint4* p = a.Wt + ((((size_t)(strip >> 1) * n_half + (F >> 2)) * 2 + (strip & 1)) * 4 + (F & 3)) * 64 + (wg & 1) * 16 + u + 32 * (q & 1);
        return kf < kf_real ? p : a.zeros + lane;
    };
    u32x4_t w[RKF][4];
#pragma unroll
    for (int i = 0; i < RKF; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) w[i][g] = __builtin_bit_cast(u32x4_t, ld_matrix<NKF>(w_addr(g, LKF > 0 ? i / 3 * 4 + i % 3 : i)));
#pragma unroll
    for (int i = 0; i < RKF; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (i * 4 + g < RKF * 4 - 36) asm volatile("" : "+a"(w[i][g]));
    for (int i = 0; i < LKF; ++i) {
        uint4 v[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) v[g] = ld_matrix<NKF>(w_addr(g, 4 * i + 3));
#pragma unroll
        for (int g = 0; g < 4; ++g) wl[(i * 4 + g) * 64] = v[g];
    }
    if (tid == 0) {
        const unsigned gone = __hip_atomic_load(a.aborted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned seen = 0;
        for (unsigned looks = 0;; ++looks) {
            seen = __hip_atomic_load(a.sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (gone) seen |= LEAVE;
            if ((seen & LEAVE) || seen == a.expect) break;
            if (looks >= a.arrive_looks) {
                unsigned old = seen;
                if (__hip_atomic_compare_exchange_strong(a.sync, &old, seen | LEAVE, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    seen |= LEAVE;
                    __hip_atomic_fetch_add(a.aborted, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // the one workgroup that decides it
                    break;
                }
                continue;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        *go = (seen & LEAVE) ? 0u : 1u;
    }
    __syncthreads();
    if (*go == 0u) return;

    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void*)a.xchg, 0, 64 * h, 0x00020000);
    const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc((void*)la.xprev, 0, 64 * h, 0x00020000);
    const int cu = tid & 15, cc = tid >> 4;            // cell: unit and column of this thread
    const size_t unit = (size_t)16 * wg + cu;
    const size_t H = h;
    unsigned limit = a.spin_limit;
    int l_at = la.l0;
    for (int s = 0; s < la.n_lvl; ++s) {
        const int n = la.rows[s], np = s > 0 ? la.rows[s - 1] : 0;
        // this lane's column of the operand: row u of the level (lanes beyond the level repeat row 0), its predecessor's column
        const int my_t = la.tab.lvl_rows[l_at + (u < n ? u : 0)];
        int col = u < n ? u : 0;
        if (s > 0) {
            const int want = la.tab.lpred[a.r0 + my_t] - a.r0;
            col = 0;
            for (int i = 0; i < np; ++i) if (la.tab.lvl_rows[l_at - np + i] == want) col = i;
        }
        const unsigned ph = (((s - 1) >> 1) & 1) ? 0u : TAG;
        // 8-value vector 4 kf + q of this wavefront's quarter, at this lane's column
        const int cols = s > 0 ? 16 : 32;
        const __amdgpu_buffer_rsrc_t brs = s > 0 ? xrs : prs;
        const unsigned mine0 = (unsigned)((s > 0 ? ((s - 1) & 1) * h * 32 : 0) + ((wave * (h >> 5) + q) * cols + col) * 16);
        auto fetch = [&](int gr, u32x4_t (&d)[GF]) {
#pragma unroll
            for (int j = 0; j < GF; ++j) {
                const int kf = gr * GF + j;
                d[j] = __builtin_amdgcn_raw_buffer_load_b128(brs, mine0, (kf < kf_real ? kf : 0) * 64 * cols, SC1);
            }
        };
        floatx4 acc[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
        u32x4_t b[2][GF], wb[4];
        fetch(0, b[0]);
#pragma unroll
        for (int gr = 0; gr < NKF / GF; ++gr) {
            if (s > 0) {
                for (unsigned looks = 0;; ++looks) {
                    asm volatile("" ::: "memory");
                    unsigned off = 0u;
#pragma unroll
                    for (int j = 0; j < GF; ++j) off |= (b[gr & 1][j].x ^ ph) | (b[gr & 1][j].y ^ ph) | (b[gr & 1][j].z ^ ph) | (b[gr & 1][j].w ^ ph);
                    if (__all((off & TAG) == 0u)) break;
                    if (looks >= limit) {
                        limit = 0;
                        if (lane == 0) __hip_atomic_store(a.fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        break;
                    }
                    fetch(gr, b[gr & 1]);
                }
            }
            if (gr + 1 < NKF / GF) fetch(gr + 1, b[(gr + 1) & 1]);
            if constexpr (LKF > 0) {
#pragma unroll
                for (int g = 0; g < 4; ++g) wb[g] = *(const u32x4_t*)&wl[(gr * 4 + g) * 64];
            }
            auto plain = [&](unsigned x) {
                x ^= ph;
                const unsigned over = ((x & 0x7fff7fffu) + 0x407f407fu) & 0x80008000u;
                return x | (over >> 1);
            };
            if (s > 0) {
#pragma unroll
                for (int j = 0; j < GF; ++j) {
                    u32x4_t& v = b[gr & 1][j];
                    v.x = plain(v.x); v.y = plain(v.y); v.z = plain(v.z); v.w = plain(v.w);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < GF; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const u32x4_t wv = (LKF > 0 && j == 3) ? wb[g] : w[LKF > 0 ? (gr * 3 + j) % RKF : gr * GF + j][g];
                    acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wv), __builtin_bit_cast(bf16x8_t, b[gr & 1][j]), acc[g], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) *(floatx4*)(part + ((wave * 4 + g) * 16 + u) * 16 + 4 * q) = acc[g];   // column u, units 4q..
        __builtin_amdgcn_sched_barrier(0);   // what the cell needs is requested here: above it would take registers from the weights
        const bool cell = cc < n;
        const int ct = la.tab.lvl_rows[l_at + (cell ? cc : 0)], cr = a.r0 + ct;
        float gin[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) gin[g] = a.g_in[(size_t)ct * 4 * H + g * H + unit] + a.bias[g * H + unit];
        const float cp = a.state[((size_t)la.tab.lpred[cr] * 2 + 1) * H + unit];   // this workgroup's own store of the level before, or older
        __syncthreads();
        float pre[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            float v = part[(g * 16 + cc) * 16 + cu];
#pragma unroll
            for (int w_ = 1; w_ < 4; ++w_) v += part[((w_ * 4 + g) * 16 + cc) * 16 + cu];
            pre[g] = v + gin[g];
        }
        const float cn = lstm_gate(pre[1], false) * cp + lstm_gate(pre[0], false) * lstm_gate(pre[2], true);
        const float hn = lstm_gate(pre[3], false) * lstm_gate(cn, true);
        const __bf16 hb = (__bf16)hn;
        const unsigned mine = __builtin_bit_cast(uint16_t, hb), other = (unsigned)__shfl_xor((int)mine, 1);
        const unsigned pair = mine | (other << 16);   // even threads: units cu, cu + 1
        if (cell) {
            if ((cu & 1) == 0) {
                if (s + 1 < la.n_lvl)
                    __builtin_amdgcn_raw_buffer_store_b32((pair & ~TAG) | (((s >> 1) & 1) ? 0u : TAG), xrs,
                                                          (unsigned)(((s & 1) * h * 32) + (((int)unit >> 3) * 16 + cc) * 16 + ((int)unit & 7) * 2), 0, SC1);
                if (a.xnext) *(unsigned*)((char*)a.xnext + ((unit >> 3) * a.Tp + ct) * 16 + (unit & 7) * 2) = pair;
            }
            a.state[((size_t)cr * 2) * H + unit] = hn;
            a.state[((size_t)cr * 2 + 1) * H + unit] = cn;
        }
        if (la.x) {   // a strip's statistics are the sum of two workgroups', in either order the same
            const float xg = hn * la.gain[unit], xg_next = __shfl_xor(xg, 1);
            float ssq = hn * hn;
            ssq += __shfl_xor(ssq, 1);
            ssq += __shfl_xor(ssq, 2);
            ssq += __shfl_xor(ssq, 4);
            ssq += __shfl_xor(ssq, 8);
            if (cell) {
                la.x[((unit >> 2) * a.Tp + ct) * 4 + (unit & 3)] = hn;
                if ((cu & 1) == 0) *(unsigned*)((char*)la.xb + ((unit >> 3) * a.Tp + ct) * 16 + (unit & 7) * 2) = pack_bf16x2(xg, xg_next);
                if (cu == 0) __hip_atomic_fetch_add(la.ssq + (unit >> 5) * a.Tp + ct, ssq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();   // part is written again, and the next level reads this one's cell states
        l_at += n;
    }
}

// What LAYER 1 leaves for the decoder block, for rows whose states are there: the residual stream x, x * gain and the
// per-strip sums of squares (the second half of k_lstm_cell).
struct LstmOutArgs { const float* state; float* x; void* xb; const float* gain; float* ssq; int r0, n, rows, Tp, h; };   // rows n .. rows-1: zeros
template <typename EL>
static __global__ __launch_bounds__(256) void k_lstm_out(LstmOutArgs a) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int qn = a.h / 4;
    const int t = (int)(idx / qn);
    const int f0 = (int)(idx % qn) * 4;
    if (t >= a.rows) return;               // whole strips leave together: h is a multiple of 64
    const float4 v = t < a.n ? *(const float4*)(a.state + (size_t)(a.r0 + t) * 2 * a.h + f0) : make_float4(0.f, 0.f, 0.f, 0.f);
    ((float4*)a.x)[(size_t)(f0 >> 2) * a.Tp + t] = v;
    const float4 gn = *(const float4*)(a.gain + f0);
    store4_act<EL>(a.xb, a.Tp, f0, t, v.x * gn.x, v.y * gn.y, v.z * gn.z, v.w * gn.w);
    float ssq = v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    ssq += __shfl_xor(ssq, 1);
    ssq += __shfl_xor(ssq, 2);
    ssq += __shfl_xor(ssq, 4);
    if ((f0 & 31) == 0) a.ssq[(size_t)(f0 >> 5) * a.Tp + t] = ssq;
}
