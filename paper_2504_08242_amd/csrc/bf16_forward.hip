// Orchestration of the bf16 (matrix-core) path: one stage forward over one sub-sequence with its
// cached prefix (Jupiter paper, Sec. IV-A.2); decoder layer of Sec. II-A in its Llama-2 form.
//
// One launch that prepares the call (norm of the first layer, rotary table; bf16_misc.hip), then per layer, up to 16 rows,
// five launches on one stream (the caller's):
//   QKV GEMM (+ rotary + KV append)  ->  chunk attention  ->  O projection (+ residual)  ->  gate/up GEMM (+ SwiGLU)
//   ->  down projection (+ residual)
// and seven (the first norm is the preparing launch's) for more rows (the caller's stream, or a lane's of the multi-chunk call):
//   reduce+norm  ->  QKV GEMM (+ rotary + KV append)  ->  chunk attention  ->  O GEMM (K-split partials)
//   ->  reduce+norm  ->  gate/up GEMM (+ SwiGLU)  ->  down GEMM (K-split partials)
// The projections back to d_model are too narrow to fill 256 CUs with tall tiles, so they split K and
// write fp32 partial tiles; the next reduce+norm pass adds them to the fp32 residual stream in a fixed
// order (bitwise reproducible) on its way to the normalised bf16 rows it has to produce anyway.
#include "w4_plan.h"

namespace jup {

hipError_t bf16_pack_weights(const jup_stage& st, const jup_layer_weights_t* layers, hipStream_t s) {
    const jup_stage_config_t& c = st.cfg;
    const size_t d = c.d_model;
    hipError_t e = gemm_configure();
    if (e == hipSuccess) e = rows_configure();
    if (e == hipSuccess) e = attention_configure();
    if (e != hipSuccess) return e;
    for (int l = 0; l < c.n_layers; ++l) {
        char* base = (char*)st.packed + (size_t)l * st.pl.layer_bytes;
        const jup_layer_weights_t& w = layers[l];
        launch_pack_qkv((u16*)(base + st.pl.wqkv), (const u16*)w.wq, (const u16*)w.wk, (const u16*)w.wv, c.d_model, s);
        launch_pack_gate_up((u16*)(base + st.pl.wgu), (const u16*)w.w_gate, (const u16*)w.w_up, c.d_model, c.d_ffn, s);
        launch_pack_plain((u16*)(base + st.pl.wo), (const u16*)w.wo, c.d_model, c.d_model, s);
        launch_pack_plain((u16*)(base + st.pl.wdown), (const u16*)w.w_down, c.d_model, c.d_ffn, s);
        e = hipMemcpyAsync(base + st.pl.g_attn, w.g_attn, d * 2, hipMemcpyDeviceToDevice, s);
        if (e == hipSuccess) e = hipMemcpyAsync(base + st.pl.g_mlp, w.g_mlp, d * 2, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

// 4-bit stage: codes and scales of the seven matrices go into their packed layouts (w4_gemm.hip); gains as above.
// A stage created with w4_expanded also gets their bf16 values in the layouts of the bf16 stage.
hipError_t w4_pack_weights(const jup_stage& st, const jup_layer_weights_t* layers, hipStream_t s) {
    const jup_stage_config_t& c = st.cfg;
    const size_t d = c.d_model;
    hipError_t e = attention_configure();
    if (e == hipSuccess) e = w4_wide_configure();
    if (e == hipSuccess && c.w4_expanded) e = gemm_configure();
    if (e != hipSuccess) return e;
    for (int l = 0; l < c.n_layers; ++l) {
        char* base = (char*)st.packed + (size_t)l * st.pl.layer_bytes;
        const jup_layer_weights_t& w = layers[l];
        launch_pack_w4_qkv((unsigned char*)(base + st.pl.wqkv), (float*)(base + st.pl.sqkv), w.wq, w.wk, w.wv, w.sq, w.sk,
                           w.sv, c.d_model, s);
        launch_pack_w4_gate_up((unsigned char*)(base + st.pl.wgu), (float*)(base + st.pl.sgu), w.w_gate, w.w_up, w.s_gate,
                               w.s_up, c.d_model, c.d_ffn, s);
        launch_pack_w4_plain((unsigned char*)(base + st.pl.wo), (float*)(base + st.pl.so), w.wo, w.so, c.d_model,
                             c.d_model, s);
        launch_pack_w4_plain((unsigned char*)(base + st.pl.wdown), (float*)(base + st.pl.sdown), w.w_down, w.s_down,
                             c.d_model, c.d_ffn, s);
        if (c.w4_expanded) {
            launch_expand_qkv((u16*)(base + st.pl.xqkv), w.wq, w.wk, w.wv, w.sq, w.sk, w.sv, c.d_model, s);
            launch_expand_gate_up((u16*)(base + st.pl.xgu), w.w_gate, w.w_up, w.s_gate, w.s_up, c.d_model, c.d_ffn, s);
            launch_expand_plain((u16*)(base + st.pl.xo), w.wo, w.so, c.d_model, c.d_model, s);
            launch_expand_plain((u16*)(base + st.pl.xdown), w.w_down, w.s_down, c.d_model, c.d_ffn, s);
        }
        e = hipMemcpyAsync(base + st.pl.g_attn, w.g_attn, d * 2, hipMemcpyDeviceToDevice, s);
        if (e == hipSuccess) e = hipMemcpyAsync(base + st.pl.g_mlp, w.g_mlp, d * 2, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

// bt == nullptr: one chunk of n tokens at position pos of cache kv.
// bt != nullptr: bt->n_branches chunks of bt->n_tok tokens each, n = their total number of rows; the rows of
// branch b are appended to and attend over cache bt->kv[b] from position bt->pos0[b] (pos and kv are unused).
// Everything that is not attention or cache traffic sees one [n, d] activation matrix either way, so the
// stage's weights are streamed once for all branches.
// link != nullptr: scratch buffer and cross-stream events of a chunk that overlaps with its neighbours.
// tree != nullptr (host table, bt == nullptr): the n tokens are a token tree; only the rotary positions
// (pos + depth) and the mask inside the chunk differ from an ordinary chunk.
hipError_t bf16_forward(const jup_stage& st, const void* hidden_in, int n, int pos, const KvView& kv,
                        void* hidden_out, hipStream_t s, const BranchTable* bt, const TreeTable* tree,
                        const ChunkLink* link) {
    const jup_stage_config_t& c = st.cfg;
    const int d = c.d_model, f = c.d_ffn, H = c.n_heads;
    char* ws = (char*)(link && link->workspace ? link->workspace : st.workspace);
    float* x32 = (float*)(ws + st.wl.x32);
    u16* xn = (u16*)(ws + st.wl.xn);
    u16* q = (u16*)(ws + st.wl.q);
    u16* o = (u16*)(ws + st.wl.o);
    u16* act = (u16*)(ws + st.wl.act);
    float* partial = (float*)(ws + st.wl.partial);
    float2* rope = (float2*)(ws + st.wl.rope);
    // 1 / rms of the rows (branches of up to 16 tokens): lives from a reduce + norm pass to the projection behind it, when nothing is in o
    float* factor = (float*)(ws + st.wl.o);
    const size_t split_stride = (size_t)n * d;

    if (c.n_layers == 0) return hipMemcpyAsync(hidden_out, hidden_in, (size_t)n * d * 2, hipMemcpyDeviceToDevice, s);
    const BranchTable* bt_dev = nullptr;
    const TreeTable* tree_dev = nullptr;
    const AttScratch att{(float*)(ws + st.wl.att_split), (int*)(ws + st.wl.att_count), st.wl.att_split_rows,
                         st.wl.att_count_n};
    const bool shared = link != nullptr;                    // other chunks' kernels run beside this chunk's
    const bool rows = n <= kMaxProjectRows && !shared;      // (see `project` below)
    int max_keys = 0;  // batched branches: the longest key range
    double keys = (double)pos + n;  // read per layer
    {
        TraceScope ts(st, JUP_K_RMSNORM, s);
        // (more than 16 rows: the first reduce + norm pass reads hidden_in again, half the bytes of an fp32 copy that nothing else
        // would read.  The three launches of this kind of a one-layer call, which writes no x32 behind its last projection
        // either: 2048 rows of d_model 4096 67.5 -> 60.3 us, 512 rows 29.1 -> 27.0)
        const BeginArgs a{rows ? x32 : nullptr, (const u16*)hidden_in, (const u16*)((const char*)st.packed + st.pl.g_attn), xn, n, d, c.rms_eps,
                          rope, c.rope_theta, att.split_count, (int)att.counters};
        if (bt) {
            bt_dev = (const BranchTable*)(ws + st.wl.branches);
            launch_begin_branches(a, *bt, (BranchTable*)(ws + st.wl.branches), s);
            keys = 0;  // (a shared prefix once)
            for (int b = 0; b < bt->n_branches; ++b) {
                const int end = bt->pos0[b] + bt->n_tok;
                max_keys = end > max_keys ? end : max_keys;
                keys += end - (b > 0 ? bt->kv[b].n_shared : 0);
            }
        } else if (tree) {
            tree_dev = (const TreeTable*)(ws + st.wl.tree);
            launch_begin_tree(a, pos, *tree, (TreeTable*)(ws + st.wl.tree), s);
        } else {
            launch_begin_chunk(a, pos, s);
        }
    }

    // 4-bit stage: the projections read codes, everything else is the bf16 path.  With the expanded copy at hand,
    // chunks beyond one pass of the 4-bit kernels (64 rows) take the bf16 projections on it.
    const bool expanded = c.dtype == JUP_BF16_W4 && c.w4_expanded && n > 64;
    const bool w4 = c.dtype == JUP_BF16_W4 && !expanded;
    const size_t wqkv = expanded ? st.pl.xqkv : st.pl.wqkv, wo = expanded ? st.pl.xo : st.pl.wo;
    const size_t wgu = expanded ? st.pl.xgu : st.pl.wgu, wdown = expanded ? st.pl.xdown : st.pl.wdown;
    // Weights (bf16, or codes and scales), keys and values a call goes through, against the 256 MB of the last-level cache.
    const double layer_bytes = (w4 ? 17.0 / 32 : 2.0) * (4.0 * d * d + 3.0 * d * f) + 512.0 * H * keys;
    const bool from_memory = c.n_layers * layer_bytes > 256e6;
    // Back to d_model.  Calls of up to 16 rows: the O / down projections finish the residual and the rows of the next
    // projection themselves (row_gemm.hip); their sums of squares take the place of the partial sums in the workspace.  All
    // other calls leave partial sums to the reduce + norm pass; batches of branches of up to 16 tokens in a form that gives
    // every branch the bits it has alone: bf16 weights up to max_split_rows, codes whatever the rows.  (The bf16 copy of a
    // 4-bit stage is not what a branch of up to 64 rows runs on alone.)
    const bool small_branches = !rows && bt && bt->n_tok <= kMaxProjectRows && (w4 || (!expanded && n <= max_split_rows(d)));
    const bool as_rows = rows || small_branches;
    const int n_tok = bt ? bt->n_tok : n;
    const int splits_o = w4 ? w4_partial_splits(n_tok, d, d) : as_rows ? row_splits(d) : gemm_plan_splits(n, d, d, shared);
    const int splits_down = w4 ? w4_partial_splits(n_tok, d, f) : as_rows ? row_splits(d) : gemm_plan_splits(n, d, f, shared);
    float* late_factor = small_branches ? factor : nullptr;
    float* ssq = partial;
    // back to d_model: in [n, k] times w; gain: of the norm that follows (null behind the last layer)
    auto project = [&](const u16* in, const void* w, const void* w_scale, int k, const u16* gain) {
        if (rows || (small_branches && !w4)) {
            RowArgs a{};
            a.A = in; a.W = w; a.w_scale = (const float*)w_scale; a.M = n; a.N = d; a.K = k;
            a.splits = k == d ? splits_o : splits_down;
            a.x32 = x32; a.gain = gain; a.xn = xn; a.ssq = ssq; a.out = gain ? nullptr : (u16*)hidden_out;
            a.partial = partial;
            return rows ? launch_project_rows(w4, a, s) : launch_project_split(a, s);
        }
        GemmArgs a{};
        a.A = in; a.W = (const u16*)w; a.w_scale = (const float*)w_scale; a.M = n; a.N = d; a.K = k;
        a.n_tok = n_tok; a.partial = partial; a.shared_gpu = shared;
        return w4 ? launch_gemm_w4(EPI_PARTIAL, a, s) : launch_gemm_partial(a, s);
    };
    hipError_t e = hipSuccess;
    for (int l = 0; l < c.n_layers && e == hipSuccess; ++l) {
        const char* wb = (const char*)st.packed + (size_t)l * st.pl.layer_bytes;
        const u16* g1 = (const u16*)(wb + st.pl.g_attn);
        const u16* g2 = (const u16*)(wb + st.pl.g_mlp);
        if (l > 0 && !rows) {
            TraceScope ts(st, JUP_K_RMSNORM, s);
            launch_reduce_norm(x32, nullptr, partial, splits_down, split_stride, g1, xn, late_factor, nullptr, n, d, c.rms_eps, s);
        }
        {
            TraceScope ts(st, JUP_K_GEMM_QKV, s);
            GemmArgs a{};
            a.A = xn; a.W = (const u16*)(wb + wqkv); a.M = n; a.N = 3 * d; a.K = d; a.n_tok = n_tok;
            a.q_out = q; a.rope = rope; a.kv = kv; a.layer = l; a.n_heads = H; a.d_model = d; a.pos0 = pos;
            a.branches = bt_dev;
            a.shared_gpu = shared;
            a.ssq = rows && l > 0 ? ssq : nullptr; a.rms_eps = c.rms_eps;
            a.row_factor = l > 0 ? late_factor : nullptr;
            a.w_scale = (const float*)(wb + st.pl.sqkv);
            e = w4 ? launch_gemm_w4(EPI_QKV, a, s) : launch_gemm_qkv(a, s);
        }
        // keys and values of this layer are in the cache: the next chunk may attend to them; this chunk needs
        // those of the chunk before it
        if (link && link->record_qkv && e == hipSuccess) e = hipEventRecord(link->record_qkv[l], s);
        for (int w = 0; link && w < link->n_wait && e == hipSuccess; ++w) e = hipStreamWaitEvent(s, link->wait_qkv[w][l], 0);
        {
            TraceScope ts(st, JUP_K_ATTENTION, s);
            if (e != hipSuccess) break;
            if (bt) e = launch_branch_attention(q, o, bt->n_tok, bt->n_branches, d, H, bt_dev, max_keys, l, s, att, from_memory);
            else e = launch_chunk_attention(q, o, n, d, H, pos, kv, l, s, att, from_memory, tree_dev, shared);
        }
        {
            TraceScope ts(st, JUP_K_GEMM_O, s);
            if (e == hipSuccess) e = project(o, wb + wo, wb + st.pl.so, d, g2);
        }
        if (!rows) {
            TraceScope ts(st, JUP_K_RMSNORM, s);
            launch_reduce_norm(x32, l == 0 ? (const u16*)hidden_in : nullptr, partial, splits_o, split_stride, g2, xn, late_factor, nullptr, n, d, c.rms_eps, s);
        }
        {
            TraceScope ts(st, JUP_K_GEMM_GATE_UP, s);
            GemmArgs a{};
            a.A = xn; a.W = (const u16*)(wb + wgu); a.M = n; a.N = 2 * f; a.K = d; a.n_tok = n_tok; a.act = act; a.shared_gpu = shared;
            a.ssq = rows ? ssq : nullptr; a.rms_eps = c.rms_eps;
            a.row_factor = late_factor;
            a.w_scale = (const float*)(wb + st.pl.sgu);
            if (e == hipSuccess) e = w4 ? launch_gemm_w4(EPI_SWIGLU, a, s) : launch_gemm_swiglu(a, s);
        }
        {
            TraceScope ts(st, JUP_K_GEMM_DOWN, s);
            const u16* next_g = l + 1 < c.n_layers ? (const u16*)(wb + st.pl.layer_bytes + st.pl.g_attn) : nullptr;
            if (e == hipSuccess) e = project(act, wb + wdown, wb + st.pl.sdown, f, next_g);
        }
    }
    if (e != hipSuccess || rows) return e;
    // last layer's down-projection partials + residual -> hidden_out
    launch_reduce_norm(x32, nullptr, partial, splits_down, split_stride, nullptr, nullptr, nullptr, (u16*)hidden_out, n, d,
                       c.rms_eps, s);
    return hipGetLastError();
}

}  // namespace jup
