// A long commit of a bf16 drafter: up to FV_DRAFT_WIDE_ROWS pairs through the drafter in one pass (included by fv_step.hip).
// What bounds it.  A pass of up to 256 rows reads every matrix of the drafter for itself and its reductions besides (about 430 us at the 7B
// width), one of up to 64 rows the same matrices again (390), and each starts its chain launches by reading the recurrent matrices (27 us a layer).
// Here the products serve all rows, in the tiles of a long prompt (k_gemm_ring, WIDE: whole K ranges, no partial tiles), and one chain launch
// a layer runs over all of them.  The head's logits are looked at for values that are no numbers where they are computed, and stored
// only for the rows whose lists are wanted: the last `keep`, which stay open as the phase's rows 0 .. keep-1, and the k-1 in front of those, whose
// outputs the phase's first levels may come from.
#pragma once

// input rows z = [feature ; embedding], 32 rows x 32 features a workgroup; rows beyond m are zero
struct WideBeginArgs {
    const int32_t* tok;       // [m]
    const float* ext;         // [m][h]
    const void* table;        // embedding [V][h]
    void* xz;                 // [2h/8][ld][8]
    float* ones;              // [ld] factors of the products without a norm
    uint32_t* chain; int chain_words;   // exchange area of the chain launches to clear
    int m, ld, h;
};
static __global__ __launch_bounds__(256) void k_wide_begin(WideBeginArgs a) {
    const int tid = threadIdx.x, flat = blockIdx.y * gridDim.x + blockIdx.x;
    for (int i = flat * 256 + tid; i < a.chain_words; i += gridDim.x * gridDim.y * 256) a.chain[i] = 0u;
    const int t = blockIdx.y * 32 + (tid >> 3), f0 = blockIdx.x * 32 + (tid & 7) * 4;   // eight lanes read 128 bytes of a row
    if (blockIdx.x == 0 && tid < 32) a.ones[blockIdx.y * 32 + tid] = 1.f;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (t < a.m) {
        if (f0 < a.h) {
            const float4 x = *(const float4*)(a.ext + (size_t)t * a.h + f0);
            v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        } else {
            const uint2 u = *(const uint2*)((const uint16_t*)a.table + (size_t)a.tok[t] * a.h + (f0 - a.h));
            const uint4 w = make_uint4(u.x, u.y, 0u, 0u);
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = Tr<BF16>::at(w, c);
        }
    }
    store4_act<BF16>(a.xz, a.ld, f0, t, v[0], v[1], v[2], v[3]);
}

// The states behind the last row, of both layers: the phase's last open row continues from them, and so does the next commit.  Not if the pass
// came to nothing (a chain launch that left, values that are no numbers): the call then runs its pieces one by one.
struct WideStateArgs { const float* from[2]; float* state[2]; const int32_t* bad; int32_t* bad_out; int last, keep, h; };
static __global__ __launch_bounds__(256) void k_wide_state(WideStateArgs a) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx < 3) { a.bad_out[idx] = a.bad[idx]; __threadfence_system(); }
    if (idx >= 2 * a.h || a.bad[0] || a.bad[2]) return;
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        const float v = a.from[l][(size_t)a.last * 2 * a.h + idx];
        a.state[l][(size_t)(a.keep - 1) * 2 * a.h + idx] = v;
        a.state[l][(size_t)FV_MAX_TREE * 2 * a.h + idx] = v;
    }
}

// m rows (65 .. wide.P) whose tokens are in d->h_tok and whose features are the rows of `ext`, from slot d->L on
template <typename EL, int D>
int run_draft_wide(fv_drafter* d, const float* ext, int m, int keep) {
    if constexpr (Tr<EL>::E != 8) {
        return FV_E_BAD_ARG;
    } else {
        fv_ctx* c = d->core;
        const fv_cfg& cf = c->cfg;
        const Layout& ly = c->lay;
        const DraftLayout& dl = d->lay;
        const DraftWide& w = dl.wide;
        const int h = cf.hidden, ld = (int)rup(m, 256), first = m - keep, n_hist = std::min(d->k - 1, first);
        hipStream_t st = c->stream;
        if (m < 1 || keep < 1 || keep > m || keep > FV_MAX_TREE || ld > w.P) return FV_E_BAD_ARG;
        char* const base = c->arena + ly.off_stage;
        auto at = [&](size_t off) { return base + off; };
        HIPCHK(hipMemcpyAsync(at(w.tok), d->h_tok, (size_t)m * 4, hipMemcpyHostToDevice, st));
        {
            WideBeginArgs ba;
            ba.tok = (const int32_t*)at(w.tok); ba.ext = ext; ba.table = d->target->arena + d->target->lay.off_embed; ba.xz = at(w.xz);
            ba.ones = (float*)at(w.ones); ba.chain = d->at<uint32_t>(dl.off_chain); ba.chain_words = (256 + 8 * h) / 4;
            ba.m = m; ba.ld = ld; ba.h = h;
            hipLaunchKernelGGL(k_wide_begin, dim3(2 * h / 32, ld / 32), dim3(256), 0, st, ba);
            PromptIngestArgs ia;
            ia.T = m; ia.Tp = ld; ia.L = d->L; ia.half_d = D / 2; ia.log2_base = std::log2((double)cf.rope_base);
            ia.mask = (uint64_t*)at(w.mask); ia.rope_cs = (float2*)at(w.rope);
            PadArgs pa = k_padding<EL>(c, 0, 0, 0, ld);
            const size_t offs[3] = {w.xb, w.attn, w.act};
            const GemmPlan* plans[3] = {&ly.gm[GM_QKV], &ly.gm[GM_O], &ly.gm[GM_DN]};
            for (int i = 0; i < 3; ++i) pa.p[i] = (uint4*)(at(offs[i]) + (size_t)plans[i]->K * ld * 2);
            hipLaunchKernelGGL(k_ingest_prompt, dim3(ld / 4 + pad_blocks(pa)), dim3(256), 0, st, ia, pa);
            HIPCHK(hipGetLastError());
        }
        ManyRows rows;
        rows.m = m; rows.ld = ld; rows.L = d->L;
        rows.x = (float*)at(w.x); rows.ssq = (float*)at(w.ssq); rows.rinv = (float*)at(w.rinv);
        rows.xb = at(w.xb); rows.q = at(w.q); rows.qlo = at(w.qlo); rows.attn = at(w.attn); rows.act = at(w.act);
        rows.mask = (const uint64_t*)at(w.mask); rows.rope = (const float2*)at(w.rope);
        float* const ones = (float*)at(w.ones);
        for (int layer = 0; layer < 2; ++layer) {
            GemmArgs ga = many_args(rows, layer == 0 ? dl.ih0.gm : dl.hh.gm, d->arena + dl.off_w[2 * layer], at(layer == 0 ? w.xz : w.xh), ones);
            ga.logits = (float*)at(w.gin); ga.Vpad = 4 * h;
            hipLaunchKernelGGL((k_gemm_commit<D, EPI_LOGITS>), many_grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
            HIPCHK(hipGetLastError());
            ChainRows cr;
            cr.n = m; cr.Tp = ld; cr.r0 = 0; cr.g_in = (const float*)at(w.gin); cr.state = (float*)at(w.state[layer]); cr.xnext = layer == 0 ? at(w.xh) : nullptr;
            const int rc = launch_lstm_chain(d, cr, layer);
            if (rc) return rc;
        }
        LstmOutArgs oa;
        oa.state = (const float*)at(w.state[1]); oa.x = (float*)at(w.x); oa.xb = at(w.xb); oa.gain = c->gain(0); oa.ssq = (float*)at(w.ssq);
        oa.r0 = 0; oa.n = m; oa.rows = ld; oa.Tp = ld; oa.h = h;
        hipLaunchKernelGGL((k_lstm_out<EL>), dim3((unsigned)(((size_t)(h / 4) * ld + 255) / 256)), dim3(256), 0, st, oa);
        HIPCHK(hipGetLastError());

        const int rc = run_many_layer<EL, D>(c, rows, 0, false, d->at<float>(dl.off_ones));   // the decoder block
        if (rc) return rc;
        {
            GemmArgs ga = many_args(rows, ly.gm[GM_LM], d->target->arena + d->target->lay.off_lm, rows.xb, ones);
            ga.logits = d->at<float>(dl.off_logits); ga.Vpad = ly.Vpad;
            ga.L = first; ga.Hq = n_hist; ga.Hkv = cf.vocab; ga.tickets = d->at<int>(dl.off_bad);   // see EPI_HEAD
            hipLaunchKernelGGL((k_gemm_commit<D, EPI_HEAD>), many_grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
            HIPCHK(hipGetLastError());
        }
        TopmArgs ta;
        ta.logits = d->at<float>(dl.off_logits); ta.top_tok = d->at<int32_t>(dl.off_top_tok); ta.top_val = d->at<float>(dl.off_top_val);
        ta.bad = d->at<int32_t>(dl.off_bad); ta.gate = ta.bad;
        ta.r0 = 0; ta.n = keep; ta.V = cf.vocab; ta.Vpad = ly.Vpad; ta.m = FV_DRAFT_MMAX;
        DraftOutArgs da;
        da.x = (const float*)at(w.x) + (size_t)4 * first; da.fout = d->at<float>(dl.off_fout); da.r0 = 0; da.n = keep; da.Tp = ld; da.h = h;
        hipLaunchKernelGGL(k_topm, dim3(2 * keep), dim3(FV_TOPM_THREADS), 0, st, ta, da);
        if (n_hist > 0) {   // (first >= k - 1, as the host chooses m and keep)
            ta.logits += (size_t)FV_MAX_TREE * ly.Vpad; ta.r0 = da.r0 = FV_MAX_TREE; ta.n = da.n = n_hist;
            da.x = (const float*)at(w.x) + (size_t)4 * (first - n_hist);
            hipLaunchKernelGGL(k_topm, dim3(2 * n_hist), dim3(FV_TOPM_THREADS), 0, st, ta, da);
        }
        WideStateArgs wa;
        for (int l = 0; l < 2; ++l) { wa.from[l] = (const float*)at(w.state[l]); wa.state[l] = d->state(l); }
        wa.bad = d->at<int32_t>(dl.off_bad); wa.bad_out = d->h_out + FV_MAX_TREE; wa.last = m - 1; wa.keep = keep; wa.h = h;
        hipLaunchKernelGGL(k_wide_state, dim3((2 * h + 255) / 256), dim3(256), 0, st, wa);
        HIPCHK(hipGetLastError());
        return FV_OK;
    }
}
