// Many prompt rows at once (included by fv_step.hip): the layers of a decoder pass over m consecutive rows whose only result is
// their K and V.  A chunk of max_tree rows reads every matrix for itself and leaves most of a matrix-core cycle unused;
// here the weights serve up to 2048 rows, in tiles that a workgroup computes over the whole K range (k_gemm_ring, WIDE), and
// the attention runs on pieces of 256 rows of the same buffers.
#pragma once

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

        auto args = [&](int which, const void* Wt, size_t x_off) {
            const GemmPlan& p = ly.gm[which];
            GemmArgs ga;
            memset(&ga, 0, sizeof(ga));
            ga.Wt = (const uint4*)Wt; ga.X = c->at<uint4>(x_off); ga.NG = p.NG; ga.NB = p.NB; ga.T = m; ga.ld = ld; ga.n_strips = p.n_strips;
            ga.rinv_out = c->at<float>(ly.off_prinv);
            return ga;
        };
        auto rinv = [&]() -> int {
            PhaseTimer pt(c, FV_PH_OTHER);
            RinvArgs ra;
            ra.ssq = c->at<float>(ly.off_pssq); ra.rinv = c->at<float>(ly.off_prinv); ra.n_ssq = h / 32; ra.ld = ld; ra.inv_h = 1.f / (float)h; ra.eps = cf.rms_eps;
            hipLaunchKernelGGL(k_rinv, dim3(ld / 64), dim3(256), 0, st, ra);
            HIPCHK(hipGetLastError());
            return FV_OK;
        };
        auto grid = [&](const GemmArgs& ga) { return dim3(8u * (unsigned)std::min((ga.NG + 7) / 8 * (ld / 256), 32)); };   // one workgroup per compute unit at most
        for (int l = 0; l < cf.n_layers; ++l) {
            int rc = rinv();
            if (rc) return rc;
            {
                PhaseTimer pt(c, FV_PH_GEMM);
                GemmArgs ga = args(GM_QKV, c->layer_w(l, 0), ly.off_pxb);
                ga.q_out = c->at<void>(ly.off_pq); ga.q_lo_out = c->at<void>(ly.off_pqlo); ga.kcache = c->kc(l); ga.vcache = c->vc(l);
                ga.rope_cs = c->at<float2>(ly.off_prope); ga.Hq = cf.n_q_heads; ga.Hkv = cf.n_kv_heads; ga.L = L; ga.S_pad = ly.S_pad;
                hipLaunchKernelGGL((k_gemm_ring<8, D, EPI_QKV, true>), grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
                HIPCHK(hipGetLastError());
            }
            if (l + 1 == cf.n_layers) break;   // nothing reads the last layer's rows: their K and V are what is wanted
            {
                PhaseTimer pt(c, FV_PH_ATTN);
                AttnArgs aa;
                aa.q = c->at<uint4>(ly.off_pq); aa.q_lo = c->at<uint4>(ly.off_pqlo); aa.kc = (const uint4*)c->kc(l); aa.vc = (const uint4*)c->vc(l);
                aa.out = c->at<void>(ly.off_pattn); aa.mask = c->at<uint64_t>(ly.off_pmask);
                aa.Tp = 256; aa.ld = ld; aa.pieces = ld / 256; aa.T = m; aa.TK = m; aa.L = L; aa.Hq = cf.n_q_heads; aa.Hkv = cf.n_kv_heads; aa.S_pad = ly.S_pad;
                aa.scale = 1.f / std::sqrt((float)D);
                aa.ks = 1; aa.part = nullptr; aa.tickets = nullptr;   // more pieces than one: no key split, hence no partial triples
                rc = launch_attn<EL, D>(aa, cf.n_q_heads * 8, ld / 256, st);
                if (rc) return rc;
            }
            {
                PhaseTimer pt(c, FV_PH_GEMM);
                GemmArgs ga = args(GM_O, c->layer_w(l, 1), ly.off_pattn);
                ga.x_in = ga.x = c->at<float>(ly.off_px); ga.xb = c->at<void>(ly.off_pxb); ga.gain_next = c->gain(2 * l + 1); ga.ssq_out = c->at<float>(ly.off_pssq);
                hipLaunchKernelGGL((k_gemm_ring<8, D, EPI_RESID, true>), grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
                HIPCHK(hipGetLastError());
            }
            rc = rinv();
            if (rc) return rc;
            {
                PhaseTimer pt(c, FV_PH_GEMM);
                GemmArgs ga = args(GM_GU, c->layer_w(l, 2), ly.off_pxb);
                ga.act = c->at<void>(ly.off_pact);
                hipLaunchKernelGGL((k_gemm_ring<8, D, EPI_SWIGLU, true>), grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
                HIPCHK(hipGetLastError());
            }
            {
                PhaseTimer pt(c, FV_PH_GEMM);
                GemmArgs ga = args(GM_DN, c->layer_w(l, 3), ly.off_pact);
                ga.x_in = ga.x = c->at<float>(ly.off_px); ga.xb = c->at<void>(ly.off_pxb); ga.gain_next = c->gain(2 * (l + 1)); ga.ssq_out = c->at<float>(ly.off_pssq);
                hipLaunchKernelGGL((k_gemm_ring<8, D, EPI_RESID, true>), grid(ga), dim3(FV_RING_THREADS), ring_smem(8), st, ga);
                HIPCHK(hipGetLastError());
            }
        }
        return FV_OK;
    }
}
