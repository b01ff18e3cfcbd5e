// Many rows at once (included by fv_step.hip): a decoder layer over m consecutive rows, of a prompt (below) or of a drafter's long commit
// (fv_draft_wide.hpp); and a prompt's layers, whose only result is the rows' K and V.  A chunk of max_tree rows reads every matrix for itself and leaves most of a matrix-core cycle unused;
// here the weights serve up to 2048 rows, in tiles that a workgroup computes over the whole K range (k_gemm_ring, WIDE), and
// the attention runs on pieces of 256 rows of the same buffers.
#pragma once

// The rows' buffers and where they stand: activations as in a step, rows of ld (a multiple of 256), from cache slot L on
struct ManyRows {
    int m, ld, L;
    float *x, *ssq, *rinv;
    void *xb, *q, *qlo, *attn, *act;
    const uint64_t* mask;
    const float2* rope;
};

// arguments of a product over whole K ranges
inline GemmArgs many_args(const ManyRows& b, const GemmPlan& p, const void* Wt, const void* X, float* factors) {
    GemmArgs ga;
    memset(&ga, 0, sizeof(ga));
    ga.Wt = (const uint4*)Wt; ga.X = (const uint4*)X; ga.NG = p.NG; ga.NB = p.NB; ga.T = b.m; ga.ld = b.ld; ga.n_strips = p.n_strips;
    ga.rinv_out = factors;
    return ga;
}
inline dim3 many_grid(const GemmArgs& ga) { return dim3(8u * (unsigned)std::min((ga.NG + 7) / 8 * (ga.ld / 256), 32)); }   // one workgroup per compute unit at most

// Layer l.  only_kv: nothing reads its rows, their K and V are what is wanted.  gain_next: of the norm behind it.
template <typename EL, int D>
int run_many_layer(fv_ctx* c, const ManyRows& b, int l, bool only_kv, const float* gain_next) {
    const fv_cfg& cf = c->cfg;
    const Layout& ly = c->lay;
    hipStream_t st = c->stream;
    auto rinv = [&]() -> int {
        PhaseTimer pt(c, FV_PH_OTHER);
        RinvArgs ra;
        ra.ssq = b.ssq; ra.rinv = b.rinv; ra.n_ssq = cf.hidden / 32; ra.ld = b.ld; ra.inv_h = 1.f / (float)cf.hidden; ra.eps = cf.rms_eps;
        hipLaunchKernelGGL(k_rinv, dim3(b.ld / 64), dim3(256), 0, st, ra);
        HIPCHK(hipGetLastError());
        return FV_OK;
    };
    auto resid = [&](int which, int wi, const void* X, const float* gain) -> int {
        PhaseTimer pt(c, FV_PH_GEMM);
        GemmArgs ga = many_args(b, ly.gm[which], c->layer_w(l, wi), X, b.rinv);
        ga.x_in = ga.x = b.x; ga.xb = b.xb; ga.gain_next = gain; ga.ssq_out = b.ssq;
        hipLaunchKernelGGL((k_gemm_ring<8, D, EPI_RESID, true>), many_grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
        HIPCHK(hipGetLastError());
        return FV_OK;
    };
    int rc = rinv();
    if (rc) return rc;
    {
        PhaseTimer pt(c, FV_PH_GEMM);
        GemmArgs ga = many_args(b, ly.gm[GM_QKV], c->layer_w(l, 0), b.xb, b.rinv);
        ga.q_out = b.q; ga.q_lo_out = b.qlo; ga.kcache = c->kc(l); ga.vcache = c->vc(l);
        ga.rope_cs = b.rope; ga.Hq = cf.n_q_heads; ga.Hkv = cf.n_kv_heads; ga.L = b.L; ga.S_pad = ly.S_pad;
        hipLaunchKernelGGL((k_gemm_ring<8, D, EPI_QKV, true>), many_grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
        HIPCHK(hipGetLastError());
    }
    if (only_kv) return FV_OK;
    {
        PhaseTimer pt(c, FV_PH_ATTN);
        AttnArgs aa;
        aa.q = (const uint4*)b.q; aa.q_lo = (const uint4*)b.qlo; aa.kc = (const uint4*)c->kc(l); aa.vc = (const uint4*)c->vc(l);
        aa.out = b.attn; aa.mask = b.mask;
        aa.Tp = 256; aa.ld = b.ld; aa.pieces = b.ld / 256; aa.T = b.m; aa.TK = b.m; aa.L = b.L; aa.Hq = cf.n_q_heads; aa.Hkv = cf.n_kv_heads; aa.S_pad = ly.S_pad;
        aa.scale = 1.f / std::sqrt((float)D);
        aa.ks = 1; aa.part = nullptr; aa.tickets = nullptr;   // more pieces than one: no key split, hence no partial triples
        rc = launch_attn<EL, D>(aa, cf.n_q_heads * 8, b.ld / 256, st);
        if (rc) return rc;
    }
    rc = resid(GM_O, 1, b.attn, c->gain(2 * l + 1));
    if (rc) return rc;
    rc = rinv();
    if (rc) return rc;
    {
        PhaseTimer pt(c, FV_PH_GEMM);
        GemmArgs ga = many_args(b, ly.gm[GM_GU], c->layer_w(l, 2), b.xb, b.rinv);
        ga.act = b.act;
        hipLaunchKernelGGL((k_gemm_ring<8, D, EPI_SWIGLU, true>), many_grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
        HIPCHK(hipGetLastError());
    }
    return resid(GM_DN, 3, b.act, gain_next);
}

template <typename EL, int D>
int run_prompt(fv_ctx* c, const int32_t* h_tok, int m) {
    if constexpr (Tr<EL>::E != 8) {
        return FV_E_BAD_ARG;   // fp32 prompts go chunk by chunk (lay.Pm is 0)
    } else {
        const fv_cfg& cf = c->cfg;
        const Layout& ly = c->lay;
        const int h = cf.hidden, ld = (int)rup(m, 256), L = c->cur_len;
        hipStream_t st = c->stream;
        if (m < 1 || ld > ly.Pm) return FV_E_BAD_ARG;
        HIPCHK(hipMemcpyAsync(c->at<int32_t>(ly.off_ptok), h_tok, (size_t)m * 4, hipMemcpyHostToDevice, st));
        HIPCHK(hipEventRecord(c->ev0, st));
        {
            PhaseTimer pt(c, FV_PH_OTHER);
            PromptIngestArgs ia;
            ia.T = m; ia.Tp = ld; ia.L = L; ia.half_d = D / 2; ia.log2_base = std::log2((double)cf.rope_base);
            ia.mask = c->at<uint64_t>(ly.off_pmask); ia.rope_cs = c->at<float2>(ly.off_prope);
            const PadArgs pa = k_padding<EL>(c, ly.off_pxb, ly.off_pattn, ly.off_pact, ld);
            hipLaunchKernelGGL(k_ingest_prompt, dim3(ld / 4 + pad_blocks(pa)), dim3(256), 0, st, ia, pa);
            EmbedArgs ea;
            ea.table = c->at<void>(ly.off_embed); ea.tok = c->at<int32_t>(ly.off_ptok); ea.gain = c->gain(0);
            ea.x = c->at<float>(ly.off_px); ea.xb = c->at<void>(ly.off_pxb); ea.ssq_part = c->at<float>(ly.off_pssq);
            ea.h = h; ea.T = m; ea.Tp = ld;
            hipLaunchKernelGGL((k_embed<EL>), dim3(h / 32, ld / 256), dim3(256), 0, st, ea);
            HIPCHK(hipGetLastError());
        }

        ManyRows b;
        b.m = m; b.ld = ld; b.L = L;
        b.x = c->at<float>(ly.off_px); b.ssq = c->at<float>(ly.off_pssq); b.rinv = c->at<float>(ly.off_prinv);
        b.xb = c->at<void>(ly.off_pxb); b.q = c->at<void>(ly.off_pq); b.qlo = c->at<void>(ly.off_pqlo); b.attn = c->at<void>(ly.off_pattn); b.act = c->at<void>(ly.off_pact);
        b.mask = c->at<uint64_t>(ly.off_pmask); b.rope = c->at<float2>(ly.off_prope);
        for (int l = 0; l < cf.n_layers; ++l) {
            const int rc = run_many_layer<EL, D>(c, b, l, l + 1 == cf.n_layers, c->gain(2 * (l + 1)));
            if (rc) return rc;
        }
        return FV_OK;
    }
}
