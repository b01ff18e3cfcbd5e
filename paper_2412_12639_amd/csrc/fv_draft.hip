// Host side of the drafting-phase entry points declared in include/falcon_verify.h: arena layout of
// the drafter, weight upload, the plan of a phase over a static tree (which rows each pass has, what
// they take in, which row generates which node) and the read-back helpers.  The kernel sequence of a
// pass lives in fv_draft_step.hpp (compiled with the fv_step.hip units).
#include "fv_host.hpp"
#include "fv_draft_kernels.hpp"
#include "fv_lstm_chain.hpp"

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

namespace {

enum { T_FEAT = 0, T_TOKNODE, T_TOKVAL, T_PRED, T_LPRED, T_BLOCK, T_POS, T_LVL, T_NODEGEN, T_NODERANK, T_EXP };

fv_cfg core_cfg(const fv_cfg& t) {
    fv_cfg c = t;
    c.n_layers = 1;
    c.max_tree = FV_MAX_TREE;
    return c;
}

int lstm_chain_size(int h);

// Buffers of a long commit: byte offsets inside the core context's staging area.  bf16 drafters whose recurrence runs in chain launches and whose
// matrices the ring kernel can address.
DraftWide plan_wide(const fv_cfg& t, const Layout& core, const GemmPlan& ih0, const GemmPlan& hh) {
    DraftWide w;
    bool ok = t.dtype == FV_BF16 && t.max_seq > 256 && lstm_chain_size(t.hidden) != 0 && gemm_ring_takes(ih0.NG, ih0.NB) && gemm_ring_takes(hh.NG, hh.NB);
    for (int i = 0; i < GM_COUNT; ++i) ok = ok && gemm_ring_takes(core.gm[i].NG, core.gm[i].NB);
    if (!ok) return w;
    const size_t P = w.P = (int)std::min(rup(t.max_seq, 256), (size_t)FV_DRAFT_WIDE_ROWS);
    const size_t h = t.hidden, qd = (size_t)t.n_q_heads * t.head_dim;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t r = o; o = rup(o + bytes, 256); return r; };
    w.tok = take(P * 4);
    w.xz = take((size_t)ih0.Kpad * P * 2);
    w.xh = take((size_t)hh.Kpad * P * 2);
    w.gin = take(P * 4 * h * 4);
    for (size_t& s : w.state) s = take(P * 2 * h * 4);
    w.x = take(h * P * 4);
    w.xb = take((size_t)core.gm[GM_QKV].Kpad * P * 2);
    w.q = take(qd * P * 2);
    w.qlo = take(qd * P * 2);
    w.attn = take((size_t)core.gm[GM_O].Kpad * P * 2);
    w.act = take((size_t)core.gm[GM_DN].Kpad * P * 2);
    w.ssq = take(h / 32 * P * 4);
    w.rinv = take(P * 4);
    w.ones = take(P * 4);
    w.rope = take(P * (t.head_dim / 2) * 8);
    w.mask = take(256 * 4 * 8);
    w.bytes = o;
    return w;
}

// What the staging area has to hold: the largest tensor (lstm0.w_ih) and a long commit's buffers
size_t draft_stage_elems(const fv_cfg& t, int n_wg) {
    const size_t lstm = (size_t)4 * t.hidden * 2 * t.hidden;
    if (t.dtype != FV_BF16) return lstm;
    Layout core;
    make_layout(core_cfg(t), n_wg, core, false, lstm);
    GemmPlan ih0, hh, gd, gp;
    bool ok;
    plan_gemm_forms(ih0, gd, gp, ok, (int)(4 * t.hidden / 32), (int)(2 * t.hidden), core.E, n_wg);
    plan_gemm_forms(hh, gd, gp, ok, (int)(4 * t.hidden / 32), (int)t.hidden, core.E, n_wg);
    return std::max(lstm, (plan_wide(t, core, ih0, hh).bytes + 1) / 2);
}

void make_draft_layout(const fv_cfg& t, int n_wg, DraftLayout& L) {
    const fv_cfg cc = core_cfg(t);
    Layout core;
    make_layout(cc, n_wg, core, false, draft_stage_elems(t, n_wg));
    const size_t h = t.hidden, ESZ = core.ESZ, Tpm = FV_MAX_TREE;
    plan_gemm_forms(L.ih0.gm, L.ih0.gd, L.ih0.gp, L.ih0.paired_ok, (int)(4 * h / 32), (int)(2 * h), core.E, n_wg);
    plan_gemm_forms(L.hh.gm, L.hh.gd, L.hh.gp, L.hh.paired_ok, (int)(4 * h / 32), (int)h, core.E, n_wg);
    L.wide = plan_wide(t, core, L.ih0.gm, L.hh.gm);
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t r = o; o = rup(o + bytes, 256); return r; };
    L.off_core = take(core.total);
    L.core_bytes = core.total;
    L.off_w[0] = take(L.ih0.gm.tiled_bytes);
    for (int i = 1; i < 4; ++i) L.off_w[i] = take(L.hh.gm.tiled_bytes);
    L.off_bias = take(2 * 4 * h * 4);
    L.off_ones = take(h * 4);
    L.off_xz = take((size_t)L.ih0.gm.Kpad * Tpm * ESZ);
    L.off_xh = take((size_t)L.hh.gm.Kpad * Tpm * ESZ);
    L.off_xprev = take((size_t)L.hh.gm.Kpad * Tpm * ESZ);
    L.off_gin = take(Tpm * 4 * h * 4);
    L.off_grec = take(Tpm * 4 * h * 4);
    L.state_layer_bytes = rup((size_t)(FV_MAX_TREE + 1) * 2 * h * 4, 256);
    L.off_state = take(2 * L.state_layer_bytes);
    L.off_fout = take((size_t)FV_DRAFT_OUT_ROWS * h * 4);
    L.off_top_tok = take((size_t)FV_DRAFT_OUT_ROWS * FV_DRAFT_MMAX * 4);
    L.off_top_val = take((size_t)FV_DRAFT_OUT_ROWS * FV_DRAFT_MMAX * 4);
    L.off_logits = take((size_t)2 * FV_MAX_TREE * core.Vpad * 4);   // a pass writes its padded row count from its first row on
    L.off_tables = take((size_t)FV_DRAFT_TABLES * FV_MAX_TREE * 4);
    L.off_bad = take(256);
    for (GemmPlan* p : {&L.ih0.gm, &L.ih0.gd, &L.ih0.gp, &L.hh.gm, &L.hh.gd, &L.hh.gp}) p->off_tab = take(plan_table_bytes(*p));
    size_t pb = std::max(core.part_bytes, std::max(plan_part_bytes(L.ih0.gm, L.ih0.gd, L.ih0.gp, Tpm), plan_part_bytes(L.hh.gm, L.hh.gd, L.hh.gp, Tpm)));
    L.part_bytes = pb;
    L.off_part = take(pb);
    int ngmax = std::max(L.ih0.gm.n_strips_pad, L.hh.gm.n_strips_pad);
    for (int i = 0; i < GM_COUNT; ++i) ngmax = std::max(ngmax, core.gm[i].n_strips_pad);
    L.ticket_bytes = (size_t)ngmax * 4;
    L.off_tickets = take(L.ticket_bytes);
    L.chain_bytes = 256 + 128 * h;   // two arrival counters 128 bytes apart, then [layer][2][h][16 columns] bf16 (a chain: one column)
    L.off_chain = take(L.chain_bytes);
    L.total = o;
}

int pass_any(fv_drafter* d, const DraftPass& ps) {
    const fv_cfg& cf = d->core->cfg;
    int rc;
    if (cf.dtype == FV_BF16) rc = cf.head_dim == 128 ? run_draft_pass<BF16, 128>(d, ps) : run_draft_pass<BF16, 64>(d, ps);
    else rc = cf.head_dim == 128 ? run_draft_pass<F32, 128>(d, ps) : run_draft_pass<F32, 64>(d, ps);
    if (rc != FV_OK) d->part_dirty = true;   // a pass that stopped half-way may leave partial tiles nobody consumed
    return rc;
}

DraftTables dev_tables(const fv_drafter* d) {
    DraftTables t;
    t.feat_src = d->tab(T_FEAT); t.tok_node = d->tab(T_TOKNODE); t.tok_val = d->tab(T_TOKVAL); t.pred = d->tab(T_PRED);
    t.lpred = d->tab(T_LPRED); t.block = d->tab(T_BLOCK); t.pos = d->tab(T_POS); t.lvl_rows = d->tab(T_LVL);
    t.node_gen = d->tab(T_NODEGEN); t.node_rank = d->tab(T_NODERANK); t.exp_list = d->tab(T_EXP);
    return t;
}

int wide_any(fv_drafter* d, const float* ext, int m, int keep) {
    const int rc = d->core->cfg.head_dim == 128 ? run_draft_wide<BF16, 128>(d, ext, m, keep) : run_draft_wide<BF16, 64>(d, ext, m, keep);
    if (rc != FV_OK) d->part_dirty = true;
    return rc;
}

// slots [slot0, slot0 + n) of a bf16 drafter's cache (see k_draft_clear_slots)
int clear_slots(fv_drafter* d, int slot0, int n) {
    const fv_cfg& cf = d->core->cfg;
    ClearSlotsArgs ca;
    ca.kcache = d->core->kc(0); ca.vcache = d->core->vc(0); ca.slot0 = slot0; ca.n = n; ca.Hkv = cf.n_kv_heads; ca.S_pad = d->core->lay.S_pad;
    const dim3 grid((unsigned)(((size_t)n * cf.n_kv_heads * cf.head_dim + 255) / 256));
    if (cf.head_dim == 128) hipLaunchKernelGGL((k_draft_clear_slots<BF16, 128>), grid, dim3(256), 0, d->core->stream, ca);
    else hipLaunchKernelGGL((k_draft_clear_slots<BF16, 64>), grid, dim3(256), 0, d->core->stream, ca);
    HIPCHK(hipGetLastError());
    return FV_OK;
}

// The first n error words (not finite, exchange fault, launches that left) to zero.  On the drafter's stream like all that sets them: the null stream's
// own fill is not ordered against a stream that does not wait for it, and the host does not wait for either.
int clear_errors(fv_drafter* d, size_t n) {
    hipLaunchKernelGGL(k_draft_fill, dim3(1), dim3(256), 0, d->core->stream, d->at<uint32_t>(d->lay.off_bad), 0u, n);
    HIPCHK(hipGetLastError());
    return FV_OK;
}

int32_t* htab(fv_drafter* d, int which) { return d->h_tab + (size_t)which * FV_MAX_TREE; }

int upload_tables(fv_drafter* d) {
    HIPCHK(hipMemcpyAsync(d->tab(0), d->h_tab, (size_t)FV_DRAFT_TABLES * FV_MAX_TREE * 4, hipMemcpyHostToDevice, d->core->stream));
    return FV_OK;
}

// Fragments per wavefront of the built chain kernel that takes hidden size h, 0 if none does.
int lstm_chain_size(int h) {
    if (h % 128 || h > 4096) return 0;
    for (int nkf : {2, 4, 8, 16, 32})
        if (h / 128 <= nkf) return nkf;
    return 0;
}

template <int NKF>
int launch_chain_t(const LstmChainArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(k_lstm_chain<NKF>, dim3(a.h / 16), dim3(256), lstm_chain_smem(NKF), st, a);
    return hipGetLastError() == hipSuccess ? FV_OK : FV_E_HIP;
}
template <int NKF>
int launch_levels_t(const LstmLevelArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(k_lstm_levels<NKF>, dim3(a.c.h / 16), dim3(256), lstm_level_smem(NKF), st, a);
    return hipGetLastError() == hipSuccess ? FV_OK : FV_E_HIP;
}
template <int NKF>
int set_chain_attr() {
    HIPCHK(hipFuncSetAttribute((const void*)k_lstm_levels<NKF>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lstm_level_smem(NKF)));
    HIPCHK(hipFuncSetAttribute((const void*)k_lstm_chain<NKF>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lstm_chain_smem(NKF)));
    return FV_OK;
}

// Whether the chain kernel takes this drafter: bf16, a hidden size whose recurrent matrix fits into the registers and LDS of
// h / 16 compute units (h up to 4096), and a device with that many.  At hidden 4096 a row then costs 1.85 us per layer instead
// of 33; wider drafters and fp32 ones stream the matrix once per row as before.
int lstm_chain_fits(const fv_cfg& c, bool& fits) {
    fits = false;
    if (c.dtype != FV_BF16 || !lstm_chain_size(c.hidden)) return FV_OK;
    int dev = 0, cus = 0;
    HIPCHK(hipGetDevice(&dev));
    HIPCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (c.hidden / 16 > cus) return FV_OK;
    int rc = FV_E_BAD_ARG;
    switch (lstm_chain_size(c.hidden)) {
        case 2: rc = set_chain_attr<2>(); break;
        case 4: rc = set_chain_attr<4>(); break;
        case 8: rc = set_chain_attr<8>(); break;
        case 16: rc = set_chain_attr<16>(); break;
        case 32: rc = set_chain_attr<32>(); break;
    }
    fits = rc == FV_OK;
    return rc;
}

}  // namespace

int launch_lstm_chain(fv_drafter* d, const ChainRows& cr, int layer) {
    ++d->chain_launches;
    fv_ctx* c = d->core;
    const DraftLayout& dl = d->lay;
    const int h = c->cfg.hidden;
    LstmChainArgs a;
    a.Wt = (const uint4*)(d->arena + dl.off_w[2 * layer + 1]); a.zeros = c->at<uint4>(c->lay.off_zeros);
    a.g_in = cr.g_in; a.bias = d->at<float>(dl.off_bias) + (size_t)layer * 4 * h; a.state = cr.state;
    a.xnext = cr.xnext;
    a.sync = d->at<uint32_t>(dl.off_chain) + 32 * layer;
    a.xchg = d->at<uint16_t>(dl.off_chain + 256) + (size_t)layer * 2 * h;
    a.fault = d->at<uint32_t>(dl.off_bad) + 1; a.aborted = d->at<uint32_t>(dl.off_bad) + 2;
    a.t0 = 0; a.r0 = cr.r0; a.n = cr.n; a.from = d->state(layer) + (size_t)FV_DRAFT_STATE_COMMITTED * 2 * h; a.Tp = cr.Tp; a.h = h;
    const bool leaves = d->chain_test >= 0 && d->chain_launches > d->chain_test;
    a.expect = (unsigned)(h / 16) + (leaves ? 1u : 0u);
    a.arrive_looks = leaves ? 2u : 4000u;   // some milliseconds
    a.spin_limit = FV_EXCHANGE_SPINS;
    if (cr.levels) {
        const DraftPass& ps = *cr.levels;
        LstmLevelArgs la;
        la.c = a;
        la.c.xchg = d->at<uint16_t>(dl.off_chain + 256) + (size_t)layer * 32 * h;
        la.tab = dev_tables(d); la.xprev = (const uint4*)cr.xprev; la.x = cr.x; la.xb = cr.xb; la.gain = cr.gain; la.ssq = cr.ssq; la.l0 = ps.l0; la.n_lvl = (int)ps.lvl_n.size();
        for (int i = 0; i < FV_DRAFT_KMAX; ++i) la.rows[i] = i < la.n_lvl ? ps.lvl_n[i] : 0;
        switch (lstm_chain_size(h)) {
            case 2: return launch_levels_t<2>(la, c->stream);
            case 4: return launch_levels_t<4>(la, c->stream);
            case 8: return launch_levels_t<8>(la, c->stream);
            case 16: return launch_levels_t<16>(la, c->stream);
            case 32: return launch_levels_t<32>(la, c->stream);
        }
        return FV_E_BAD_ARG;
    }
    switch (lstm_chain_size(h)) {
        case 2: return launch_chain_t<2>(a, c->stream);
        case 4: return launch_chain_t<4>(a, c->stream);
        case 8: return launch_chain_t<8>(a, c->stream);
        case 16: return launch_chain_t<16>(a, c->stream);
        case 32: return launch_chain_t<32>(a, c->stream);
    }
    return FV_E_BAD_ARG;
}

extern "C" {

int fv_drafter_workspace_bytes(const fv_cfg* target_cfg, size_t* out_bytes) {
    if (!out_bytes) return FV_E_BAD_ARG;
    int rc = check_cfg(target_cfg);
    if (rc) return rc;
    if (target_cfg->vocab > 32768) return FV_E_BAD_ARG;   // the top-list kernel keeps a row of logits in registers
    DraftLayout L;
    make_draft_layout(*target_cfg, n_workgroups(), L);
    *out_bytes = L.total;
    return FV_OK;
}

int fv_drafter_create(fv_ctx* target, int32_t k, void* dev_arena, size_t arena_bytes, fv_drafter** out) {
    if (!out) return FV_E_BAD_ARG;
    *out = nullptr;
    if (!target || k < 1 || k > FV_DRAFT_KMAX || !dev_arena || ((uintptr_t)dev_arena & 255)) return FV_E_BAD_ARG;
    if (target->cfg.vocab > 32768) return FV_E_BAD_ARG;
    fv_drafter* d = new (std::nothrow) fv_drafter();
    if (!d) return FV_E_BAD_ARG;
    d->target = target;
    d->k = k;
    make_draft_layout(target->cfg, n_workgroups(), d->lay);
    if (arena_bytes < d->lay.total) { delete d; return FV_E_BAD_ARG; }
    d->arena = (char*)dev_arena;
    auto fail = [&](int code) { fv_drafter_destroy(d); return code; };
    const fv_cfg cc = core_cfg(target->cfg);
    int rc = fv_create_ex(&cc, d->arena + d->lay.off_core, d->lay.core_bytes, target->stream, false, draft_stage_elems(target->cfg, n_workgroups()), &d->core);
    if (rc) return fail(rc);
    hipStream_t st = d->core->stream;
    // everything outside the core context's part of the arena starts at zero too (states, pad columns, tickets)
    const size_t z0 = d->lay.off_bias;
    if (hipMemsetAsync(d->arena + z0, 0, d->lay.total - z0, st) != hipSuccess) return fail(FV_E_HIP);
    if (hipStreamSynchronize(st) != hipSuccess) return fail(FV_E_HIP);
    {
        std::vector<float> ones(target->cfg.hidden, 1.f);
        if (hipMemcpy(d->arena + d->lay.off_ones, ones.data(), ones.size() * 4, hipMemcpyHostToDevice) != hipSuccess) return fail(FV_E_HIP);
    }
    for (GemmPlan* p : {&d->lay.ih0.gm, &d->lay.ih0.gd, &d->lay.ih0.gp, &d->lay.hh.gm, &d->lay.hh.gd, &d->lay.hh.gp}) {
        std::vector<int> tab;
        p->n_fix = build_split_tables(*p, tab);
        if (tab.size() * 4 > plan_table_bytes(*p)) return fail(FV_E_BAD_ARG);
        if (hipMemcpy(d->arena + p->off_tab, tab.data(), tab.size() * 4, hipMemcpyHostToDevice) != hipSuccess) return fail(FV_E_HIP);
    }
    for (const GemmForms* f : {&d->lay.ih0, &d->lay.hh})
        for (const GemmPlan* q : {&f->gd, &f->gp})
            if ((long long)q->NG * q->NB * (q->G + 1) >= (1LL << 31)) return fail(FV_E_BAD_ARG);
    if (d->lay.part_bytes >= ((size_t)1 << 31)) return fail(FV_E_BAD_ARG);
    d->scr.part = d->at<float>(d->lay.off_part); d->scr.part_bytes = (unsigned)d->lay.part_bytes;
    d->scr.tickets = d->at<int>(d->lay.off_tickets); d->scr.ticket_bytes = d->lay.ticket_bytes;
    d->scr.dirty = &d->part_dirty;
    {   // kernel per LSTM matrix up to 64 rows: the same rule (and the same tuning switch) as the decoder's matrices
        const int base = gemm_kind_from_env();
        d->kind_ih0 = (base == GEMM_PAIRED && !d->lay.ih0.paired_ok) ? GEMM_DIRECT : base;
        d->kind_hh = (base == GEMM_PAIRED && !d->lay.hh.paired_ok) ? GEMM_DIRECT : base;
    }
    rc = lstm_chain_fits(target->cfg, d->chain_ok);
    if (rc) return fail(rc);
    { const char* e = getenv("FV_EXCHANGE_TEST"); if (e && !strncmp(e, "chain", 5)) d->chain_test = e[5] == ':' ? atoi(e + 6) : 0; }
    if (hipHostMalloc((void**)&d->h_tab, (size_t)FV_DRAFT_TABLES * FV_MAX_TREE * 4, hipHostMallocDefault) != hipSuccess) return fail(FV_E_HIP);
    if (hipHostMalloc((void**)&d->h_out, (FV_MAX_TREE + 64) * 4, hipHostMallocDefault) != hipSuccess) return fail(FV_E_HIP);
    if (d->lay.wide.P && hipHostMalloc((void**)&d->h_tok, (size_t)d->lay.wide.P * 4, hipHostMallocDefault) != hipSuccess) return fail(FV_E_HIP);
    memset(d->h_tab, 0, (size_t)FV_DRAFT_TABLES * FV_MAX_TREE * 4);
    *out = d;
    return FV_OK;
}

void fv_drafter_destroy(fv_drafter* d) {
    if (!d) return;
    if (d->core) fv_destroy(d->core);
    if (d->h_tab) (void)hipHostFree(d->h_tab);
    if (d->h_out) (void)hipHostFree(d->h_out);
    if (d->h_tok) (void)hipHostFree(d->h_tok);
    delete d;
}

int fv_drafter_init_weights(fv_drafter* d, const fv_drafter_host_weights* w) {
    if (!d || !w) return FV_E_BAD_ARG;
    for (int l = 0; l < 2; ++l)
        if (!w->lstm_w_ih[l] || !w->lstm_w_hh[l] || !w->lstm_b[l]) return FV_E_BAD_ARG;
    const size_t h = d->core->cfg.hidden;
    int rc = init_layer_weights(d->core, 0, w->wq, w->wk, w->wv, w->wo, w->wg, w->wu, w->wd, w->g_attn, w->g_mlp);
    if (rc) return rc;
    rc = upload_tiled(d->core, d->lay.ih0.gm, d->arena + d->lay.off_w[0], w->lstm_w_ih[0], 4 * h * 2 * h, (int)(4 * h));
    if (rc) return rc;
    rc = upload_tiled(d->core, d->lay.hh.gm, d->arena + d->lay.off_w[1], w->lstm_w_hh[0], 4 * h * h, (int)(4 * h));
    if (rc) return rc;
    rc = upload_tiled(d->core, d->lay.hh.gm, d->arena + d->lay.off_w[2], w->lstm_w_ih[1], 4 * h * h, (int)(4 * h));
    if (rc) return rc;
    rc = upload_tiled(d->core, d->lay.hh.gm, d->arena + d->lay.off_w[3], w->lstm_w_hh[1], 4 * h * h, (int)(4 * h));
    if (rc) return rc;
    for (int l = 0; l < 2; ++l)
        HIPCHK(hipMemcpy(d->arena + d->lay.off_bias + (size_t)l * 4 * h * 4, w->lstm_b[l], 4 * h * 4, hipMemcpyHostToDevice));
    d->core->weights_set = true;
    d->weights_set = true;
    return fv_draft_reset(d);
}

int fv_draft_reset(fv_drafter* d) {
    if (!d) return FV_E_BAD_ARG;
    hipStream_t st = d->core->stream;
    const size_t n = 2 * d->lay.state_layer_bytes / 4;   // all LSTM states, the committed one included
    hipLaunchKernelGGL(k_draft_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d->at<uint32_t>(d->lay.off_state), 0u, n);
    if (d->cache_bad) {   // a masked key is multiplied by zero, which a value that is no number survives: none may stay in a slot beside real ones
        const Layout& ly = d->core->lay;
        const size_t nk = ly.kv_layer_bytes / 4;
        for (char* slab : {d->core->kc(0), d->core->vc(0)})
            hipLaunchKernelGGL(k_draft_fill, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, st, (uint32_t*)slab, 0u, nk);
        d->cache_bad = false;
    }
    HIPCHK(hipGetLastError());
    HIPCHK(hipStreamSynchronize(st));
    d->L = d->L0 = 0;
    d->n_chain = d->n_rows = 0;
    return FV_OK;
}

int fv_draft_commit(fv_drafter* d, const int32_t* tokens, const float* dev_features, int32_t n) {
    if (!d || !tokens || !dev_features || n < 1) return FV_E_BAD_ARG;
    if (!d->weights_set || !d->target->weights_set) return FV_E_NO_PREFILL;
    const fv_cfg& cf = d->core->cfg;
    if ((long long)d->L + n > cf.max_seq) return FV_E_CACHE_FULL;
    for (int i = 0; i < n; ++i)
        if (tokens[i] < 0 || tokens[i] >= cf.vocab) return FV_E_TOKEN_RANGE;
    hipStream_t st = d->core->stream;
    bool chains = n >= 2 && d->chain_call();
    bool merge = cf.dtype == FV_BF16;   // pieces whose last rows stay open; off once one of them came to nothing
    bool hist_done = false;
    float total_ms = 0.f;
    for (int done = 0; done < n;) {
        // What stays open as the phase's chain are the last 1 to 64 rows (so that a tree has room for its own).  fp32: pieces of 64 rows, of which those
        // are the last.  bf16: up to 256 rows go in one pass, open ones included (65 to 256 rows at the 7B width: a pass of up to 256
        // rows 430 us and another of up to 64 rows 390 before), more than 256 in wide passes of up to 1024 (fv_draft_wide.hpp).  Both sides of that line, device us
        // of the call at hidden 256 / 1024 / 2048 / 4096, the passes that it takes first: 100 rows 350 / 419 / 503 / 762 against 379 / 468 / 658 / 1024 in a wide
        // one (which multiplies 256 columns in tiles that leave compute units idle), 256 rows 757 / 876 / 1039 / 1493 against 771 / 895 / 1123 / 1642; 257 rows
        // 774 / 869 / 1111 / 1732 wide against 885 / 985 / 1209 / 1792 as 256 and one, 300 rows 883 / 981 / 1237 / 1897 against 992 / 1099 / 1334 / 1980, 512 rows
        // 1411 / 1538 / 1841 / 2707 against 1513 / 1676 / 2012 / 2949.  Where a pass came to
        // nothing -- a chain launch that left, a value that is no number, which is reported with the piece it lies in -- the call goes on with
        // pieces of 256 rows and the open ones by themselves.
        const int left = n - done, tail = (n - 1) % 64 + 1, front = left - tail;
        const bool wide = merge && left > 256 && d->lay.wide.P > 0 && chains;
        int m, keep;                             // rows of this pass, those of them that stay open
        if (wide) {
            m = std::min(left, d->lay.wide.P);
            keep = m == left ? tail : 64;
        } else if (merge && left > 64) {
            m = std::min(left, 256);
            keep = m == left ? tail : m;
        } else {
            m = front > 0 ? std::min(front, cf.dtype == FV_BF16 ? 256 : 64) : left;
            keep = m;
        }
        if (d->n_chain > 0 && d->k > 1 && !hist_done) {       // outputs of the last k-1 committed rows survive the phase that ends
            HistArgs ha;
            ha.fout = d->at<float>(d->lay.off_fout); ha.top_tok = d->at<int32_t>(d->lay.off_top_tok); ha.top_val = d->at<float>(d->lay.off_top_val);
            ha.n_prev = d->n_chain; ha.k = d->k; ha.h = cf.hidden;
            hipLaunchKernelGGL(k_draft_hist, dim3(1), dim3(256), 0, st, ha);
            HIPCHK(hipGetLastError());
        }
        hist_done = false;
        d->L0 = d->L;
        const bool cut = keep < m;
        auto tables = [&](int rows, int skip) {   // committed pairs: plain causal order
            for (int i = 0; i < rows; ++i) {
                htab(d, T_FEAT)[i] = -1 - (done + skip + i);
                htab(d, T_TOKNODE)[i] = -1;
                htab(d, T_TOKVAL)[i] = tokens[done + skip + i];
                htab(d, T_PRED)[i] = i - 1;
                htab(d, T_LPRED)[i] = i == 0 ? FV_DRAFT_STATE_COMMITTED : i - 1;
                htab(d, T_BLOCK)[i] = i;
                htab(d, T_POS)[i] = d->L0 + i;
                htab(d, T_LVL)[i] = i;
            }
        };
        int rc;
        bool took_chain = false;   // the rows' recurrence ran in chain launches
        if (wide) memcpy(d->h_tok, tokens + done, (size_t)m * 4);
        else {
            tables(m, 0);
            rc = upload_tables(d);
            if (rc) return rc;
        }
        HIPCHK(hipEventRecord(d->core->ev0, st));
        DraftPass ps;
        ps.r0 = 0; ps.n = m; ps.l0 = 0; ps.ext = dev_features; ps.commit = true;
        if (!wide) ps.lvl_n.assign(m, 1);
        // One row costs a chain launch as much as the separate launches (the matrix is read once either way).  A chain launch
        // whose workgroups did not get on the chip together has done nothing; the pass is then run again without, and the pieces behind it too.
        ps.chain = chains && m >= 2;
        for (;;) {
            took_chain = wide || ps.chain;
            rc = wide ? wide_any(d, dev_features + (size_t)done * cf.hidden, m, keep) : pass_any(d, ps);
            if (rc) return rc;
            if (!wide) {
                if (cut) {
                    DraftSliceArgs sa;
                    sa.fout = d->at<float>(d->lay.off_fout); sa.top_tok = d->at<int32_t>(d->lay.off_top_tok); sa.top_val = d->at<float>(d->lay.off_top_val);
                    sa.logits = d->at<float>(d->lay.off_logits); sa.state[0] = d->state(0); sa.state[1] = d->state(1);
                    sa.bad = d->at<int32_t>(d->lay.off_bad); sa.s = m - keep; sa.keep = keep; sa.k = d->k; sa.h = cf.hidden; sa.Vpad = d->core->lay.Vpad;
                    hipLaunchKernelGGL(k_draft_slice, dim3(keep + d->k - 1), dim3(256), 0, st, sa);
                    HIPCHK(hipGetLastError());
                }
                StateKeepArgs ka;
                ka.state0 = d->state(0); ka.state1 = d->state(1); ka.aborted = d->at<uint32_t>(d->lay.off_bad) + 2; ka.row = keep - 1; ka.h = cf.hidden;
                ka.bad = d->at<int32_t>(d->lay.off_bad); ka.bad_out = d->h_out + FV_MAX_TREE; ka.finite_only = cut ? 1 : 0;
                hipLaunchKernelGGL(k_state_keep, dim3((2 * cf.hidden + 255) / 256), dim3(256), 0, st, ka);
                HIPCHK(hipGetLastError());
            }
            HIPCHK(hipEventRecord(d->core->ev1, st));
            HIPCHK(hipStreamSynchronize(st));
            if (took_chain) d->chain_outcome(d->h_out[FV_MAX_TREE + 2]);
            if (!took_chain || !d->h_out[FV_MAX_TREE + 2] || d->h_out[FV_MAX_TREE + 1]) break;
            rc = clear_errors(d, 3);
            if (rc) return rc;
            ps.chain = chains = false;
            if (wide) {   // its block ran on states that are not there, which may be no numbers
                rc = clear_slots(d, d->L, m);
                if (rc) return rc;
                break;
            }
        }
        if (d->h_out[FV_MAX_TREE + 1]) { d->part_dirty = true; return FV_E_EXCHANGE_TIMEOUT; }
        float ms = 0.f;
        HIPCHK(hipEventElapsedTime(&ms, d->core->ev0, d->core->ev1));
        total_ms += ms;
        if (wide && !chains) { hist_done = true; continue; }   // the launches left: the same rows again, without them
        if (cut && d->h_out[FV_MAX_TREE]) {                    // not finite somewhere: which piece, and what stands before it, the small pieces say
            rc = clear_errors(d, 1);
            if (rc) return rc;
            rc = clear_slots(d, d->L, m);
            if (rc) return rc;
            merge = false; hist_done = true;
            continue;
        }
        d->L += m;
        d->n_chain = d->n_rows = keep;
        if (cut) {
            d->L0 = d->L - keep;
            tables(keep, m - keep);
        }
        done += m;
        if (d->h_out[FV_MAX_TREE]) {
            d->cache_bad = true;
            rc = clear_errors(d, 1);
            if (rc) return rc;
            return FV_E_NONFINITE;
        }
    }
    d->last_ms = total_ms;
    return FV_OK;
}

int fv_draft_tree(fv_drafter* d, const int32_t* parent, const int32_t* depth, const int32_t* rank, int32_t n_nodes, int32_t root_token,
                  int32_t* tokens_out) {
    if (!d || !parent || !depth || !rank || !tokens_out || n_nodes < 1) return FV_E_BAD_ARG;
    if (!d->weights_set) return FV_E_NO_PREFILL;
    if (d->n_chain < 1 || d->L < d->k) return FV_E_NO_PREFILL;   // a phase starts with a commit; the root block needs k committed pairs
    if (d->n_rows != d->n_chain) return FV_E_NO_PREFILL;          // one tree per phase
    if (n_nodes > FV_MAX_TREE) return FV_E_TREE_TOO_BIG;
    const fv_cfg& cf = d->core->cfg;
    const int k = d->k, n = n_nodes;
    if (parent[0] != -1) return FV_E_TREE_ORDER;
    for (int i = 1; i < n; ++i)
        if (parent[i] < 0 || parent[i] >= i) return FV_E_TREE_ORDER;
    if (depth[0] != 0) return FV_E_TREE_DEPTH;
    for (int i = 1; i < n; ++i)
        if (depth[i] != depth[parent[i]] + 1) return FV_E_TREE_DEPTH;
    for (int i = 1; i < n; ++i)
        if (rank[i] < 0 || rank[i] >= FV_DRAFT_MMAX || rank[i] >= cf.vocab) return FV_E_BAD_ARG;
    if (root_token < 0 || root_token >= cf.vocab) return FV_E_TOKEN_RANGE;

    // ---- the plan: blocks (one per node at a depth that is a multiple of k and has children), their rows, and for
    // every node the output row and rank that give its token
    std::vector<int> reach(depth, depth + n);
    for (int i = n - 1; i > 0; --i) reach[parent[i]] = std::max(reach[parent[i]], reach[i]);
    int max_depth = 0;
    for (int i = 0; i < n; ++i) max_depth = std::max(max_depth, (int)depth[i]);
    const int n_pass = (max_depth + k - 1) / k;          // the chain pass of the commit counts as the first
    std::vector<std::vector<int>> rows_of(n);            // anchor node -> output row ids of its block
    rows_of[0].resize(k);
    for (int j = 0; j < k; ++j) {                        // root block: the last k committed rows, C[n_chain - 1 + j] of [history, chain]
        const int c = d->n_chain - 1 + j;
        rows_of[0][j] = (c < k - 1) ? FV_MAX_TREE + c : c - (k - 1);
    }
    auto ancestor_at = [&](int i, int dep) { while (depth[i] > dep) i = parent[i]; return i; };
    std::vector<DraftPass> passes;
    bool any_chain = false;
    int next_row = d->n_chain, lvl_at = 0, exp_at = 0;
    int32_t *t_feat = htab(d, T_FEAT), *t_node = htab(d, T_TOKNODE), *t_val = htab(d, T_TOKVAL), *t_pred = htab(d, T_PRED),
            *t_lpred = htab(d, T_LPRED), *t_block = htab(d, T_BLOCK), *t_pos = htab(d, T_POS), *t_lvl = htab(d, T_LVL),
            *t_gen = htab(d, T_NODEGEN), *t_rank = htab(d, T_NODERANK), *t_exp = htab(d, T_EXP);
    const int base_pos = d->L - 1;                       // position of the root row (the last committed pair)
    for (int p = 1; p < n_pass; ++p) {
        DraftPass ps;
        ps.r0 = next_row; ps.l0 = lvl_at;
        std::vector<std::vector<int>> by_level(k);
        for (int a = 0; a < n; ++a) {
            if (depth[a] != p * k || reach[a] <= depth[a]) continue;
            const int rows = std::min(k, reach[a] - (int)depth[a]);
            const int up = ancestor_at(a, (p - 1) * k);
            if ((int)rows_of[up].size() < k) return FV_E_BAD_ARG;   // cannot happen: a node k levels down has a full block above it
            if (next_row + rows > FV_MAX_TREE) return FV_E_TREE_TOO_BIG;
            for (int j = 0; j < rows; ++j) {
                const int r = next_row++;
                rows_of[a].push_back(r);
                t_feat[r] = rows_of[up][j];
                t_node[r] = ancestor_at(a, (p - 1) * k + j + 1);
                t_val[r] = 0;
                const int before = (j > 0) ? r - 1 : (up == 0 ? d->n_chain - 1 : rows_of[up][k - 1]);
                t_pred[r] = before;
                t_lpred[r] = before;
                t_block[r] = FV_MAX_TREE + a;   // chain rows use their own index as block id
                t_pos[r] = base_pos + (p - 1) * k + j + 1;
                by_level[j].push_back(r - ps.r0);
            }
        }
        ps.n = next_row - ps.r0;
        if (ps.n == 0) return FV_E_BAD_ARG;   // cannot happen: a tree deeper than p*k has a node at depth p*k with children
        for (int j = 0; j < k; ++j) {
            if (by_level[j].empty()) continue;
            ps.lvl_n.push_back((int)by_level[j].size());
            for (int t : by_level[j]) t_lvl[lvl_at++] = t;
        }
        // Levels of up to 16 rows each in one launch per layer (a level's rows are a subset of the blocks of the level
        // before, so the counts never grow, which the kernel's exchange relies on).  One level too: k = 1 and a tree of 30 nodes (five passes of a level
        // each) 249 us of device time against 398 as separate launches at hidden 256, 270 / 423 at 512, 353 / 458 at 1024, 673 / 731 at 2048, 863 / 874 at 2560, 1187 / 1220 at
        // 3584, and 1369 to 1384 / 1372 at 4096, where both are the read of the matrix.
        ps.chain = d->chain_ok && ps.lvl_n.size() >= 1 && ps.lvl_n.size() <= FV_DRAFT_KMAX;
        for (size_t j = 0; j < ps.lvl_n.size(); ++j) ps.chain = ps.chain && ps.lvl_n[j] <= 16 && (j == 0 || ps.lvl_n[j] <= ps.lvl_n[j - 1]);
        any_chain = any_chain || ps.chain;
        passes.push_back(ps);
    }
    if ((long long)d->L0 + next_row > cf.max_seq) return FV_E_CACHE_FULL;
    // the list row and rank every node's token is read from (the root block's lists exist since the commit)
    for (int i = 1; i < n; ++i) {
        const int dd = depth[i], p = (dd - 1) / k, j = (dd - 1) % k;
        const int a = ancestor_at(i, p * k);
        if (j >= (int)rows_of[a].size()) return FV_E_BAD_ARG;
        t_gen[i] = rows_of[a][j];
        t_rank[i] = rank[i];
        t_exp[exp_at++] = i;
    }
    t_gen[0] = 0; t_rank[0] = 0;

    // ---- run: tokens stay on the device between passes
    hipStream_t st = d->core->stream;
    int rc = upload_tables(d);
    if (rc) return rc;
    if (any_chain && !d->chain_call()) {
        any_chain = false;
        for (DraftPass& ps : passes) ps.chain = false;
    }
    for (;;) {
        HIPCHK(hipEventRecord(d->core->ev0, st));
        for (const DraftPass& ps : passes) {
            rc = pass_any(d, ps);
            if (rc) return rc;
        }
        {   // every node's token (the passes read theirs from the top lists)
            ExpandArgs ea;
            ea.tab = dev_tables(d); ea.top_tok = d->at<int32_t>(d->lay.off_top_tok); ea.node_tok = d->h_out;
            ea.bad = d->at<int32_t>(d->lay.off_bad); ea.bad_out = d->h_out + FV_MAX_TREE;
            ea.n = exp_at;
            hipLaunchKernelGGL(k_draft_expand, dim3(1), dim3(256), 0, st, ea);
            HIPCHK(hipGetLastError());
        }
        HIPCHK(hipEventRecord(d->core->ev1, st));
        HIPCHK(hipStreamSynchronize(st));
        if (any_chain) d->chain_outcome(d->h_out[FV_MAX_TREE + 2]);
        if (!any_chain || !d->h_out[FV_MAX_TREE + 2] || d->h_out[FV_MAX_TREE + 1]) break;
        // a launch over several levels left because its workgroups were not on the chip together: the tree once more without
        rc = clear_errors(d, 3);
        if (rc) return rc;
        rc = clear_slots(d, d->L0 + d->n_chain, next_row - d->n_chain);   // (its passes ran on what the ones before had left of their inputs)
        if (rc) return rc;
        any_chain = false;
        for (DraftPass& ps : passes) ps.chain = false;
    }
    if (d->h_out[FV_MAX_TREE + 1]) { d->part_dirty = true; return FV_E_EXCHANGE_TIMEOUT; }
    HIPCHK(hipEventElapsedTime(&d->last_ms, d->core->ev0, d->core->ev1));
    d->n_rows = next_row;
    if (d->h_out[FV_MAX_TREE]) {
        d->cache_bad = true;
        rc = clear_errors(d, 1);
        if (rc) return rc;
        return FV_E_NONFINITE;
    }
    d->h_out[0] = root_token;
    for (int i = 0; i < n; ++i)
        if (d->h_out[i] < 0 || d->h_out[i] >= cf.vocab) return FV_E_HIP;   // cannot happen with finite logits
    memcpy(tokens_out, d->h_out, (size_t)n * 4);
    return FV_OK;
}

int fv_draft_get_state(fv_drafter* d, int32_t* committed, int32_t* phase_rows, int32_t* chain_rows) {
    if (!d || !committed || !phase_rows || !chain_rows) return FV_E_BAD_ARG;
    *committed = d->L;
    *phase_rows = d->n_rows;
    *chain_rows = d->n_chain;
    return FV_OK;
}

int fv_draft_get_launches(fv_drafter* d, int32_t* one_launch, int32_t* gave_up) {
    if (!d || !one_launch || !gave_up) return FV_E_BAD_ARG;
    *one_launch = d->chain_launches;
    *gave_up = d->chain_gave_up;
    return FV_OK;
}

int fv_draft_get_rows(fv_drafter* d, int32_t what, int32_t row0, int32_t n, float* out) {
    if (!d || !out || n < 1 || row0 < 0) return FV_E_BAD_ARG;
    const fv_cfg& cf = d->core->cfg;
    if (what == FV_DRAFT_FEATURES) {
        if (row0 + n > FV_DRAFT_OUT_ROWS) return FV_E_BAD_ARG;
        HIPCHK(hipMemcpy(out, d->at<float>(d->lay.off_fout) + (size_t)row0 * cf.hidden, (size_t)n * cf.hidden * 4, hipMemcpyDeviceToHost));
        return FV_OK;
    }
    if (what == FV_DRAFT_LOGITS) {
        if (row0 + n > d->n_rows) return FV_E_BAD_ARG;
        const size_t Vpad = d->core->lay.Vpad;
        HIPCHK(hipMemcpy2D(out, (size_t)cf.vocab * 4, d->at<float>(d->lay.off_logits) + (size_t)row0 * Vpad, Vpad * 4, (size_t)cf.vocab * 4, n,
                           hipMemcpyDeviceToHost));
        return FV_OK;
    }
    return FV_E_BAD_ARG;
}

int fv_draft_get_top(fv_drafter* d, int32_t row0, int32_t n, int32_t* tokens_out) {
    if (!d || !tokens_out || n < 1 || row0 < 0 || row0 + n > FV_DRAFT_OUT_ROWS) return FV_E_BAD_ARG;
    HIPCHK(hipMemcpy(tokens_out, d->at<int32_t>(d->lay.off_top_tok) + (size_t)row0 * FV_DRAFT_MMAX, (size_t)n * FV_DRAFT_MMAX * 4,
                     hipMemcpyDeviceToHost));
    return FV_OK;
}

int fv_draft_read_kv(fv_drafter* d, int32_t slot0, int32_t n, float* k_out, float* v_out) {
    if (!d) return FV_E_BAD_ARG;
    return fv_read_kv(d->core, 0, slot0, n, k_out, v_out);
}

int fv_draft_last_ms(fv_drafter* d, float* ms) {
    if (!d || !ms) return FV_E_BAD_ARG;
    *ms = d->last_ms;
    return FV_OK;
}

int fv_features_device_ptr(fv_ctx* c, const float** dev_rows) {
    if (!c || !dev_rows) return FV_E_BAD_ARG;
    *dev_rows = c->at<float>(c->lay.off_feat);
    return FV_OK;
}

}  // extern "C"
