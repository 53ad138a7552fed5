// Stage executor: turns a layer list into kernel launches on the caller's stream.
//
// forward_micro : the layers on one micro-batch with the current weights; every layer output goes
//                 into the stash slot (it is the next layer's input, the ReLU mask source and, for
//                 the last layer, what the next worker reads).
// backward      : one pass over the N micro-batches of a mini-batch group, whose stashed rows are
//                 consecutive, so every layer's gradient GEMMs run once over M rows: the sum of the
//                 weight gradient over the micro-batches is the k-loop of that GEMM.  Weights are read
//                 as they are now; activations, ReLU masks, pooling winners and the softmax error
//                 signal are the forward pass's (sections "Challenge 1" and "Challenge 2", Solution).
// update        : fused momentum step over the stage's flat parameter array.
#include "stage.h"

#include "profile.h"

#include <string.h>

#include <algorithm>
#include <initializer_list>

#include <new>
#include <vector>

namespace tmps {

static thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

// launch with optional event timing of its kernel class
#define TMPS_RUN(kc, stream, expr)                 \
    do {                                           \
        ::tmps::ProfileScope scope_((kc), (stream)); \
        TMPS_HIP(expr);                            \
    } while (0)

// the contraction launchers time their kernels themselves (per kernel, by dispatch timestamps)
#define TMPS_GEMM(expr) TMPS_HIP(expr)

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Partial results of one layer's parameter gradient that may wait for the end of the backward pass.
static constexpr size_t kLatePartBytes = size_t(16) << 20;

// A pooling layer's winners from row row0 of the stash on.
static void* winners(const tmps_stage* st, const LayerRT& L, int64_t row0) {
    return st->stash + L.aux_off + (size_t)row0 * L.out_elems * maxpool_winner_bytes(L.d.dims[3]);
}

static ConvShape conv_shape(const tmps_layer_desc& d, int B) {
    ConvShape c;
    c.B = B; c.H = d.dims[0]; c.W = d.dims[1]; c.Cin = d.dims[2]; c.Cout = d.dims[3];
    c.R = d.dims[4]; c.S = d.dims[5]; c.stride = d.dims[6]; c.pad = d.dims[7];
    c.Ho = (c.H + 2 * c.pad - c.R) / c.stride + 1;
    c.Wo = (c.W + 2 * c.pad - c.S) / c.stride + 1;
    return c;
}

static bool on16(std::initializer_list<const void*> all) {
    uintptr_t bits = 0;
    for (const void* p : all) bits |= reinterpret_cast<uintptr_t>(p);
    return (bits & 15) == 0;
}

// Whether layer i is an affine layer over the channels of the convolution that it reads.  (Layers that follow each other agree in the number of their values
// only: one may read a result as a map of other channels, and is then a launch of its own.)
static bool affine_of_conv(const tmps_stage& st, int i) {
    return i >= 1 && st.layers[i].d.kind == TMPS_AFFINE && st.layers[i].in_t == i - 1 && st.layers[i - 1].d.kind == TMPS_CONV2D &&
           st.layers[i].d.dims[2] == st.layers[i - 1].d.dims[3];
}

// ... and that convolution is 1 x 1 with unit stride
static bool pointwise_below(const tmps_stage& st, int i) {
    if (!affine_of_conv(st, i)) return false;
    const int32_t* c = st.layers[i - 1].d.dims;
    return c[4] == 1 && c[5] == 1 && c[6] == 1 && c[7] == 0;
}

// The MFMA convolutions index positions with 24 bits and tensors with 31 (larger ones take an element-wise path): a
// forward pass over several micro-batches stays within that.
static bool conv_index_range_ok(const ConvShape& c) {
    const int64_t pin = (int64_t)c.B * c.H * c.W, pout = (int64_t)c.B * c.Ho * c.Wo;
    return pin < (1 << 24) && pout < (1 << 24) && pin * c.Cin < (int64_t(1) << 31) && pout * c.Cout < (int64_t(1) << 31);
}

int stage_layout(tmps_stage& st, const tmps_layer_desc* layers, int n_layers, const tmps_stage_cfg* cfg) {
    if (!layers || !cfg || n_layers < 1) return fail(TMPS_EINVAL, "null layers/cfg or no layers");
    if (cfg->dtype != TMPS_F32 && cfg->dtype != TMPS_BF16_F32MASTER) return fail(TMPS_EINVAL, "unknown dtype %d", cfg->dtype);
    if (cfg->micro_batch < 1 || cfg->n_micro < 1) return fail(TMPS_EINVAL, "micro_batch and n_micro must be positive");
    if (cfg->n_micro > 64) return fail(TMPS_EUNSUPPORTED, "at most 64 micro-batches per mini-batch");
    if (cfg->max_stash < cfg->n_micro || cfg->max_stash % cfg->n_micro != 0)
        return fail(TMPS_EMICRO, "max_stash (%d) must be a positive multiple of n_micro (%d): a mini-batch is N equal micro-batches",
                    cfg->max_stash, cfg->n_micro);
    st.cfg = *cfg;
    st.asz = act_bytes(cfg->dtype);
    st.in_esize = st.asz;
    st.layers.clear();
    st.max_run = cfg->n_micro;
    st.ws_fwd_bytes = 0;
    const int mb = cfg->micro_batch;
    const int M = mb * cfg->n_micro;
    const int f32 = cfg->dtype == TMPS_F32 ? kWsF32 : 0;
    const int64_t rows_all = (int64_t)cfg->max_stash * mb;
    int64_t poff = 0, gmax = 0;
    size_t soff = 0, ws = 0;
    bool any_skip = false, any_join = false;
    for (int i = 0; i < n_layers; ++i) {
        LayerRT L;
        L.d = layers[i];
        const int32_t* d = L.d.dims;
        L.relu = (L.d.flags & TMPS_FLAG_RELU) != 0;
        L.act = L.relu ? 1 : ((L.d.flags & TMPS_FLAG_GELU) ? 2 : 0);
        L.in_t = i - 1;
        const int src = (L.d.flags >> 8) & 0xff;
        if (src > 1) {
            if (L.d.kind != TMPS_CONV2D) return fail(TMPS_EUNSUPPORTED, "layer %d: only a convolution can read an earlier layer's result", i);
            if (i - src < -1) return fail(TMPS_ESHAPE, "layer %d: its source lies before the stage input", i);
            L.in_t = i - src;
            any_join = true;
        }
        switch (L.d.kind) {
            case TMPS_LINEAR: {
                if (d[0] < 1 || d[1] < 1) return fail(TMPS_EINVAL, "layer %d: linear dims must be positive", i);
                if ((L.d.flags & TMPS_FLAG_RELU) && (L.d.flags & TMPS_FLAG_GELU))
                    return fail(TMPS_EINVAL, "layer %d: ReLU and GELU are exclusive", i);
                if (d[2] < 0 || d[3] < 0) return fail(TMPS_EINVAL, "layer %d: negative skip or row count", i);
                L.rps = d[3] > 0 ? d[3] : 1;
                L.skip = d[2];
                L.in_elems = (int64_t)L.rps * d[0]; L.out_elems = (int64_t)L.rps * d[1];
                L.w_count = (int64_t)d[0] * d[1]; L.b_count = d[1];
                if (L.skip) {
                    const int src = i - L.skip;
                    if (src < 0) return fail(TMPS_ESHAPE, "layer %d: residual source lies before the stage", i);
                    if (st.layers[src].d.kind != TMPS_LAYERNORM)
                        return fail(TMPS_EUNSUPPORTED, "layer %d: a residual connection must start at the input of a layer-normalisation layer", i);
                    if (st.layers[src].in_elems != L.out_elems)
                        return fail(TMPS_ESHAPE, "layer %d: residual source has %lld elements per sample, the layer output %lld", i,
                                    (long long)st.layers[src].in_elems, (long long)L.out_elems);
                    for (int j = src + 1; j < i; ++j)
                        if (st.layers[j].skip && j - st.layers[j].skip == src)
                            return fail(TMPS_EUNSUPPORTED, "layer %d: two residual connections start at the same layer", i);
                    any_skip = true;
                }
                const int64_t rf = (int64_t)mb * L.rps, rb = (int64_t)M * L.rps;
                L.ws_fwd_elems = gemm_workspace_elems(rf, d[1], d[0], f32);
                L.ws_elems = std::max({L.ws_fwd_elems, gemm_workspace_elems(rb, d[0], d[1], f32),
                                       L.part_elems = gemm_workspace_elems(d[1], d[0], rb, kWsRowSums | f32)});
                for (int r = 2; r <= cfg->n_micro; ++r)   // (micro-batches forwarded together)
                    L.ws_elems = std::max(L.ws_elems, gemm_workspace_elems(r * rf, d[1], d[0], f32));
                break;
            }
            case TMPS_CONV2D: {
                for (int k = 0; k < 7; ++k)
                    if (d[k] < 1) return fail(TMPS_EINVAL, "layer %d: conv dims must be positive", i);
                if (d[7] < 0) return fail(TMPS_EINVAL, "layer %d: negative padding", i);
                if (L.act == 2) return fail(TMPS_EUNSUPPORTED, "layer %d: GELU on a convolution is not built", i);
                ConvShape c = conv_shape(L.d, M);
                while (st.max_run > 1 && !conv_index_range_ok(conv_shape(L.d, mb * st.max_run))) --st.max_run;
                if (c.Ho < 1 || c.Wo < 1) return fail(TMPS_ESHAPE, "layer %d: empty convolution output", i);
                L.in_elems = (int64_t)c.H * c.W * c.Cin;
                L.out_elems = (int64_t)c.Ho * c.Wo * c.Cout;
                L.w_count = (int64_t)c.Cout * c.R * c.S * c.Cin; L.b_count = c.Cout;
                const int64_t kf = (int64_t)c.R * c.S * c.Cin, kd = (int64_t)c.R * c.S * c.Cout;
                L.ws_fwd_elems = gemm_workspace_elems((int64_t)mb * c.Ho * c.Wo, c.Cout, kf, f32);
                L.ws_elems = std::max({L.ws_fwd_elems,
                                       gemm_workspace_elems((int64_t)M * c.H * c.W, c.Cin, kd, f32),
                                       L.part_elems = conv_wgrad_workspace_elems(cfg->dtype, c)});
                if (c.stride == 2)   // (the input gradient may walk each position's own taps only)
                    L.ws_elems = std::max(L.ws_elems, gemm_workspace_elems((int64_t)M * c.H * c.W, c.Cin,
                                                                           (int64_t)((c.R + 1) / 2) * ((c.S + 1) / 2) * c.Cout, f32));
                if (c.stride > 1 && c.R == 1 && c.S == 1)   // (or be formed for the positions that the filter reaches alone)
                    L.ws_elems = std::max(L.ws_elems, gemm_workspace_elems((int64_t)M * c.Ho * c.Wo, c.Cin, c.Cout, f32));
                for (int r = 2; r <= cfg->n_micro; ++r)
                    L.ws_elems = std::max(L.ws_elems, gemm_workspace_elems((int64_t)r * mb * c.Ho * c.Wo, c.Cout, kf, f32));
                break;
            }
            case TMPS_MAXPOOL: {
                if (d[0] < 1 || d[1] < 1 || d[2] < 1 || d[3] < 1 || d[4] < 1 || d[5] < 0 || d[5] >= d[3] ||
                    d[3] > d[0] + 2 * d[5] || d[3] > d[1] + 2 * d[5])
                    return fail(TMPS_EINVAL, "layer %d: bad pooling dims", i);
                int Ho = (d[0] + 2 * d[5] - d[3]) / d[4] + 1, Wo = (d[1] + 2 * d[5] - d[3]) / d[4] + 1;
                L.in_elems = (int64_t)d[0] * d[1] * d[2];
                L.out_elems = (int64_t)Ho * Wo * d[2];
                L.relu = false; L.act = 0;
                break;
            }
            case TMPS_AFFINE:
                if (d[0] < 1 || d[1] < 1 || d[2] < 1) return fail(TMPS_EINVAL, "layer %d: affine dims must be positive", i);
                if (L.act == 2) return fail(TMPS_EUNSUPPORTED, "layer %d: GELU on an affine layer is not built", i);
                if (i == 0 || st.layers[i - 1].act != 0)
                    return fail(TMPS_EUNSUPPORTED, "layer %d: an affine layer must follow a layer without activation", i);
                L.in_elems = L.out_elems = (int64_t)d[0] * d[1] * d[2];
                L.w_count = d[2]; L.b_count = d[2];
                L.ws_elems = L.part_elems = affine_workspace_elems((int64_t)M * d[0] * d[1], d[2]);
                break;
            case TMPS_RESADD:
                if (d[0] < 1 || d[1] < 1 || d[2] < 1 || d[3] < 1) return fail(TMPS_EINVAL, "layer %d: bad residual join", i);
                if (L.act == 2) return fail(TMPS_EUNSUPPORTED, "layer %d: GELU on a residual join is not built", i);
                if (i == 0 || i - d[3] < -1) return fail(TMPS_ESHAPE, "layer %d: a source of the join lies before the stage input", i);
                if (st.layers[i - 1].act != 0)
                    return fail(TMPS_EUNSUPPORTED, "layer %d: the layer before a residual join must have no activation", i);
                L.in_b = i - d[3];
                L.in_elems = L.out_elems = (int64_t)d[0] * d[1] * d[2];
                any_join = true;
                break;
            case TMPS_AVGPOOL:
                if (d[0] < 1 || d[1] < 1 || d[2] < 1) return fail(TMPS_EINVAL, "layer %d: pooling dims must be positive", i);
                L.in_elems = (int64_t)d[0] * d[1] * d[2];
                L.out_elems = d[2];
                L.relu = false; L.act = 0;
                break;
            case TMPS_LAYERNORM:
                if (d[0] < 1 || d[1] < 0) return fail(TMPS_EINVAL, "layer %d: bad layer-normalisation dims", i);
                L.rps = d[1] > 0 ? d[1] : 1;
                L.in_elems = L.out_elems = (int64_t)L.rps * d[0];
                L.w_count = d[0]; L.b_count = d[0];
                L.relu = false; L.act = 0;
                L.ws_elems = L.part_elems = layernorm_workspace_elems((int64_t)M * L.rps, d[0]);
                break;
            case TMPS_ATTENTION:
                if (d[0] < 1 || d[1] < 1 || d[2] < 1 || d[1] % d[2] != 0)
                    return fail(TMPS_EINVAL, "layer %d: attention needs S, D, heads positive and D a multiple of heads", i);
                L.rps = d[0];
                L.in_elems = (int64_t)d[0] * 3 * d[1];
                L.out_elems = (int64_t)d[0] * d[1];
                L.relu = false; L.act = 0;
                L.ws_elems = attention_workspace_elems(M, d[0], d[2]);
                break;
            case TMPS_EMBEDDING:
                if (i != 0) return fail(TMPS_ESHAPE, "an embedding can only be the first layer of a stage");
                if (d[0] < 1 || d[1] < 1 || d[2] < 1) return fail(TMPS_EINVAL, "layer %d: embedding dims must be positive", i);
                L.rps = d[1];
                L.in_elems = d[1];
                L.out_elems = (int64_t)d[1] * d[2];
                L.w_count = (int64_t)d[0] * d[2]; L.b_count = (int64_t)d[1] * d[2];
                L.relu = false; L.act = 0;
                st.in_esize = 4;
                break;
            case TMPS_SOFTMAX_CE:
                if (i != n_layers - 1 || !cfg->is_last || i == 0)
                    return fail(TMPS_ESHAPE, "softmax-CE must be the last layer of the last stage, after another layer");
                if (d[0] < 1 || d[1] < 0) return fail(TMPS_EINVAL, "layer %d: classes must be positive", i);
                if (st.layers.back().d.kind != TMPS_LINEAR || st.layers.back().act != 0 || st.layers.back().skip)
                    return fail(TMPS_EUNSUPPORTED, "softmax-CE must follow a plain linear layer");
                L.rps = d[1] > 0 ? d[1] : 1;
                if (st.layers.back().rps != L.rps)
                    return fail(TMPS_ESHAPE, "softmax-CE has %d rows per sample, the layer before it %d", L.rps, st.layers.back().rps);
                L.in_elems = L.out_elems = (int64_t)L.rps * d[0];
                L.relu = false; L.act = 0;
                st.label_rps = L.rps;
                break;
            default:
                return fail(TMPS_EUNSUPPORTED, "layer %d: kind %d not built", i, L.d.kind);
        }
        if (i == 0) st.in_elems = L.in_elems;
        for (int t : {L.in_t, L.d.kind == TMPS_RESADD ? L.in_b : L.in_t}) {
            const int64_t have = t < 0 ? st.in_elems : st.layers[t].out_elems;
            if (have != L.in_elems)
                return fail(TMPS_ESHAPE, "layer %d expects %lld input elements per sample, its source gives %lld", i,
                            (long long)L.in_elems, (long long)have);
        }
        if (L.w_count) {
            L.w_off = poff;
            L.b_off = poff + L.w_count;
            poff = (int64_t)align_up((size_t)(L.b_off + L.b_count), 64);
        }
        ws = std::max(ws, L.ws_elems);
        st.ws_fwd_bytes = std::max(st.ws_fwd_bytes, L.ws_fwd_elems * 4);
        st.layers.push_back(L);
    }
    if (cfg->is_last && st.layers.back().d.kind != TMPS_SOFTMAX_CE)
        return fail(TMPS_ESHAPE, "the last stage must end in softmax-CE");
    if (cfg->is_last) st.layers[n_layers - 2].out_f32 = true;
    if (!cfg->is_last) {
        if (st.layers.back().act == 2) return fail(TMPS_EUNSUPPORTED, "a stage cannot end in a GELU layer");
    }
    st.P = poff;
    st.in_elems = st.layers.front().in_elems;
    st.out_elems = cfg->is_last ? st.layers[n_layers - 2].out_elems : st.layers.back().out_elems;

    // stash: [copied inputs] then every layer's output array over all slots, and what else the backward pass needs
    st.in_off = 0;
    if (!cfg->borrow_input) soff = align_up((size_t)rows_all * st.in_elems * st.in_esize, 256);
    for (LayerRT& L : st.layers) {
        L.out_off = soff;
        L.out_esize = L.out_f32 ? 4 : st.asz;
        soff = align_up(soff + (size_t)rows_all * L.out_elems * L.out_esize, 256);
        size_t aux = 0;
        if (L.d.kind == TMPS_SOFTMAX_CE) aux = (size_t)rows_all * L.rps * 4;                  // per-row losses
        if (L.d.kind == TMPS_LAYERNORM) aux = (size_t)rows_all * L.rps * 8;                   // (mean, 1/std) per row
        if (L.d.kind == TMPS_ATTENTION) aux = (size_t)rows_all * L.d.dims[2] * L.d.dims[0] * 4;  // log-sum-exp per head and query
        if (L.d.kind == TMPS_MAXPOOL) aux = (size_t)rows_all * L.out_elems * maxpool_winner_bytes(L.d.dims[3]);   // every window's winner
        if (aux) {
            L.aux_off = soff;
            soff = align_up(soff + aux, 256);
        }
        if (L.act == 2) {
            L.z_off = soff;
            soff = align_up(soff + (size_t)rows_all * L.out_elems * st.asz, 256);
        }
    }
    if (cfg->is_last) {
        st.lab_off = soff;
        soff = align_up(soff + (size_t)rows_all * st.label_rps * 4, 256);
    }
    st.stash_bytes = soff;

    // (a convolution whose gradients come from one pass with those of the affine layer behind it: partial results of both for every workgroup of that pass)
    for (int i = 1; i < n_layers; ++i) {
        LayerRT& C = st.layers[i - 1];
        if (!pointwise_below(st, i)) continue;
        const int64_t P = (int64_t)M * C.d.dims[0] * C.d.dims[1], O = C.d.dims[3], I = C.d.dims[2];
        if (!affine_pointwise_takes(cfg->dtype, P, (int)O, (int)I)) continue;
        const size_t slabs = (size_t)affine_pointwise_slabs(P, (int)O, (int)I);
        C.part_elems = std::max<size_t>(C.part_elems, slabs * (size_t)(O * I + O));
        st.layers[i].part_elems = std::max<size_t>(st.layers[i].part_elems, slabs * 2 * (size_t)O);
    }

    // Weight gradients that the backward pass leaves to its end, in groups of one launch each.  The gradient of such a layer's
    // result then has to last that long: it gets memory of its own, unless it is the upstream gradient or the loss's.
    std::vector<int> group;
    auto close_group = [&]() {
        int dims[kWgradGroupMax][2];
        for (size_t k = 0; k < group.size(); ++k) {
            dims[k][0] = st.layers[group[k]].d.dims[0];
            dims[k][1] = st.layers[group[k]].d.dims[1];
        }
        const int64_t elems = group.empty() ? -1 : dense_wgrad_group_elems((int64_t)M * st.layers[group[0]].rps, dims, (int)group.size());
        if (elems >= 0) {
            ws = std::max(ws, (size_t)elems);
            for (int i : group) st.layers[i].grouped = true;
        }
        group.clear();
    };
    for (int i = n_layers - 1; i >= 0; --i) {
        const LayerRT& L = st.layers[i];
        if (L.d.kind != TMPS_LINEAR || !dense_wgrad_groups(cfg->dtype, (int64_t)M * L.rps, L.d.dims[0], L.d.dims[1])) continue;
        if (!group.empty() && (L.rps != st.layers[group[0]].rps || (int)group.size() == kWgradGroupMax)) close_group();
        group.push_back(i);
    }
    close_group();

    // The gradient w.r.t. a layer's input lives in a gradient buffer, unless its memory is its own (the loss layer's is kept in the stash).
    auto kept = [&](int t) { return st.layers[t].grouped && !(t == n_layers - 1 || (cfg->is_last && t == n_layers - 2)); };
    if (!cfg->is_last && st.layers.back().relu) gmax = st.layers.back().out_elems;
    for (int i = 1; i < n_layers; ++i) {
        const LayerRT& L = st.layers[i];
        if (L.d.kind == TMPS_SOFTMAX_CE) continue;
        for (int t : {L.in_t, L.d.kind == TMPS_RESADD ? L.in_b : L.in_t})
            if (t >= 0 && !kept(t)) gmax = std::max(gmax, st.layers[t].out_elems);
    }

    // scratch: gradient buffers of M rows, two boundary-gradient buffers, fp32 workspace
    size_t o = 0;
    st.n_gbuf = any_join ? 6 : (any_skip ? 4 : 2);
    // how many layers read each result (the backward pass collects one gradient contribution per reader)
    st.readers.assign(n_layers + 1, 0);
    for (int i = 0; i < n_layers; ++i) {
        const LayerRT& L = st.layers[i];
        if (L.d.kind == TMPS_EMBEDDING) continue;
        ++st.readers[L.in_t + 1];
        if (L.d.kind == TMPS_RESADD) ++st.readers[L.in_b + 1];
        if (L.d.kind == TMPS_LINEAR && L.skip) ++st.readers[st.layers[i - L.skip].in_t + 1];
    }
    st.gbuf_bytes = align_up((size_t)M * std::max<int64_t>(gmax, 1) * st.asz, 256);
    for (int k = 0; k < st.n_gbuf; ++k) { st.gbuf_off[k] = o; o += st.gbuf_bytes; }
    st.dxout_bytes = align_up((size_t)M * st.in_elems * st.asz, 256);
    st.dxout_off[0] = o; o += st.dxout_bytes;
    st.dxout_off[1] = o; o += st.dxout_bytes;
    for (int i = 0; i < n_layers; ++i)
        if (kept(i)) {
            st.layers[i].keep_off = o;   // (not 0: the gradient buffers come first)
            o += align_up((size_t)M * st.layers[i].out_elems * st.asz, 256);
        }
    // (larger ones had better be added up while the caches hold them)
    for (LayerRT& L : st.layers) {
        if (L.grouped || L.part_elems * 4 > kLatePartBytes) L.part_elems = 0;
        if (!L.part_elems) continue;
        L.part_off = o;
        o += align_up(L.part_elems * 4, 256);
    }
    st.ws_off = o; st.ws_bytes = align_up(ws * 4, 256); o += st.ws_bytes;
    st.scratch_bytes = o;
    return TMPS_OK;
}

void* stage_dxout(tmps_stage* st, int which) { return st->scratch + st->dxout_off[which & 1]; }

float* stage_row_loss(tmps_stage* st, int slot) {
    const LayerRT& L = st->layers.back();
    return reinterpret_cast<float*>(st->stash + L.aux_off) + (size_t)slot * st->cfg.micro_batch * L.rps;
}

}  // namespace tmps

using namespace tmps;

extern "C" const char* tmps_last_error(void) { return g_err; }

extern "C" int tmps_stage_bytes(const tmps_layer_desc* layers, int n_layers, const tmps_stage_cfg* cfg,
                                size_t* param_bytes, size_t* state_bytes, size_t* stash_bytes,
                                size_t* scratch_bytes) {
    tmps_stage tmp;
    int rc = stage_layout(tmp, layers, n_layers, cfg);
    if (rc != TMPS_OK) return rc;
    if (param_bytes) *param_bytes = align_up((size_t)tmp.P * (cfg->dtype == TMPS_BF16_F32MASTER ? 6 : 4), 256);
    if (state_bytes) *state_bytes = align_up((size_t)tmp.P * 8, 256);
    if (stash_bytes) *stash_bytes = tmp.stash_bytes;
    if (scratch_bytes) *scratch_bytes = tmp.scratch_bytes;
    return TMPS_OK;
}

extern "C" int tmps_stage_create(tmps_stage** out, const tmps_layer_desc* layers, int n_layers,
                                 const tmps_stage_cfg* cfg, void* params, void* state, void* stash,
                                 void* scratch) {
    if (!out) return fail(TMPS_EINVAL, "out is null");
    *out = nullptr;
    if (!params || !state || !stash || !scratch) return fail(TMPS_EINVAL, "a device region is null");
    for (const void* p : {params, state, stash, scratch})
        if (reinterpret_cast<uintptr_t>(p) & 255) return fail(TMPS_EINVAL, "device regions must be 256-byte aligned");
    tmps_stage* st = new (std::nothrow) tmps_stage();
    if (!st) return fail(TMPS_EINVAL, "out of host memory");
    int rc = stage_layout(*st, layers, n_layers, cfg);
    if (rc != TMPS_OK) {
        delete st;
        return rc;
    }
    st->params = (char*)params; st->state = (char*)state; st->stash = (char*)stash; st->scratch = (char*)scratch;
    st->master = (float*)params;
    st->wcopy = cfg->dtype == TMPS_BF16_F32MASTER ? (void*)(st->params + (size_t)st->P * 4) : nullptr;
    st->mom = (float*)state;
    st->grad = st->mom + st->P;
    st->slot_used.assign(cfg->max_stash, 0);
    st->slot_x.assign(cfg->max_stash, nullptr);
    *out = st;
    return TMPS_OK;
}

extern "C" void tmps_stage_destroy(tmps_stage* stage) { delete stage; }

extern "C" int64_t tmps_stage_param_count(const tmps_stage* stage) { return stage ? stage->P : 0; }

extern "C" int tmps_stage_param_offset(const tmps_stage* stage, int layer, int which, int64_t* offset,
                                       int64_t* count) {
    if (!stage || layer < 0 || layer >= (int)stage->layers.size() || (which != 0 && which != 1))
        return fail(TMPS_EINVAL, "bad stage, layer or selector");
    const LayerRT& L = stage->layers[layer];
    if (offset) *offset = which ? L.b_off : L.w_off;
    if (count) *count = which ? L.b_count : L.w_count;
    return TMPS_OK;
}

extern "C" int64_t tmps_stage_input_elems(const tmps_stage* stage) { return stage ? stage->in_elems : 0; }
extern "C" int64_t tmps_stage_output_elems(const tmps_stage* stage) { return stage ? stage->out_elems : 0; }
extern "C" long tmps_stage_version(const tmps_stage* stage) { return stage ? stage->version : -1; }

static size_t params_region_bytes(const tmps_stage& st) {
    return align_up((size_t)st.P * (st.cfg.dtype == TMPS_BF16_F32MASTER ? 6 : 4), 256);
}

extern "C" int tmps_stage_set_shadow(tmps_stage* stage, void* shadow, size_t bytes, int n_versions) {
    if (!stage) return fail(TMPS_EINVAL, "stage is null");
    if (n_versions < 0 || (n_versions > 0 && !shadow)) return fail(TMPS_EINVAL, "shadow region is null or n_versions negative");
    if (reinterpret_cast<uintptr_t>(shadow) & 255) return fail(TMPS_EINVAL, "the shadow region must be 256-byte aligned");
    const size_t one = params_region_bytes(*stage);
    if (bytes < one * (size_t)n_versions)
        return fail(TMPS_EINVAL, "%d versions of %zu bytes need %zu bytes, got %zu", n_versions, one, one * (size_t)n_versions, bytes);
    for (char u : stage->slot_used)
        if (u) return fail(TMPS_ESLOT, "a stash slot is in use");
    stage->shadow = n_versions ? (char*)shadow : nullptr;
    stage->shadow_n = n_versions;
    stage->param_bytes = one;
    stage->shadow_ver.assign((size_t)n_versions, -1L);
    return TMPS_OK;
}

extern "C" int tmps_stage_set_version(tmps_stage* stage, long version) {
    if (!stage) return fail(TMPS_EINVAL, "stage is null");
    if (version < 0) return fail(TMPS_EINVAL, "version %ld is negative", version);
    for (char u : stage->slot_used)
        if (u) return fail(TMPS_ESLOT, "a stash slot is in use: the version is restored between mini-batches");
    stage->version = version;
    std::fill(stage->shadow_ver.begin(), stage->shadow_ver.end(), -1L);   // kept copies belong to the old numbering
    return TMPS_OK;
}

extern "C" int tmps_stage_sync_params(tmps_stage* stage, void* hip_stream) {
    if (!stage) return fail(TMPS_EINVAL, "stage is null");
    if (stage->wcopy) TMPS_HIP(cast_f32_to_bf16(stage->master, stage->wcopy, stage->P, (hipStream_t)hip_stream));
    return TMPS_OK;
}

extern "C" void* tmps_stage_output_ptr(const tmps_stage* stage, int slot) {
    if (!stage || slot < 0 || slot >= stage->cfg.max_stash) return nullptr;
    const LayerRT& L = stage->cfg.is_last ? stage->layers[stage->layers.size() - 2] : stage->layers.back();
    return stage->out_ptr(L, (int64_t)slot * stage->cfg.micro_batch);
}

// what layer li reads: the stage input (x0, rows from row0 on) or the stashed output of the layer before it
// Runs `work` (which launches kernels on stream s and nothing else) either directly or, on a stage that replays
// graphs, as a captured graph: the first call with a key runs directly (one-off argument sets are never captured, and
// every kernel's first-launch set-up happens outside a capture), the second is captured, instantiated and launched,
// later ones launch the instantiated graph.  While per-kernel timing is on, and on the default stream, everything
// runs directly.
std::shared_mutex& tmps::capture_lock() {
    static std::shared_mutex m;
    return m;
}

template <class Work> static int run_or_replay(tmps_stage* st, const tmps_stage::GraphKey& key, hipStream_t s, Work&& work) {
    if (!st->use_graphs || s == nullptr || profile_on()) return work();   // (the default stream cannot be captured)
    auto it = st->graphs.find(key);
    if (it != st->graphs.end()) {
        TMPS_HIP(hipGraphLaunch(it->second, s));
        return TMPS_OK;
    }
    if (st->graph_seen.size() > 4096) st->graph_seen.clear();   // addresses that never repeat: forget them
    if (++st->graph_seen[key] < 2) return work();
    hipGraph_t graph = nullptr;
    int rc;
    hipError_t e;
    {
        std::unique_lock<std::shared_mutex> alone(capture_lock());
        TMPS_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        rc = work();
        e = hipStreamEndCapture(s, &graph);
    }
    if (rc != TMPS_OK || e != hipSuccess || !graph) {
        if (graph) (void)hipGraphDestroy(graph);
        if (rc != TMPS_OK) return rc;
        return fail(TMPS_EHIP, "hipStreamEndCapture failed: %s", hipGetErrorString(e));
    }
    hipGraphExec_t exec = nullptr;
    const hipError_t ei = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (ei != hipSuccess) return fail(TMPS_EHIP, "hipGraphInstantiate failed: %s", hipGetErrorString(ei));
    st->graph_seen.erase(key);
    st->graphs[key] = exec;
    TMPS_HIP(hipGraphLaunch(exec, s));
    return TMPS_OK;
}

extern "C" int tmps_stage_use_graphs(tmps_stage* st, int on) {
    if (!st) return fail(TMPS_EINVAL, "stage is null");
    st->use_graphs = on != 0;
    return TMPS_OK;
}

static bool overlap(const void* a, size_t na, const void* b, size_t nb) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
    return p && q && p < q + nb && q < p + na;
}

static const void* layer_input(const tmps_stage* st, int li, const void* x0, int64_t row0) {
    return li == 0 ? x0 : (const void*)st->out_ptr(st->layers[li - 1], row0);
}

extern "C" int tmps_forward_micro(tmps_stage* st, int slot, const void* x, void* y, const int32_t* labels,
                                  float* loss_out, void* hip_stream) {
    if (!st) return fail(TMPS_EINVAL, "stage or x is null");
    return forward_with_workspace(st, slot, 1, x, y, labels, loss_out, hip_stream, reinterpret_cast<float*>(st->scratch + st->ws_off), 0);
}

int tmps::forward_with_workspace(tmps_stage* st, int slot, int count, const void* x, void* y, const int32_t* labels,
                                 float* loss_out, void* hip_stream, float* ws, int before) {
    if (!st || !x) return fail(TMPS_EINVAL, "stage or x is null");
    if (slot < 0 || slot >= st->cfg.max_stash) return fail(TMPS_ESLOT, "slot %d outside 0..%d", slot, st->cfg.max_stash - 1);
    if (slot % st->cfg.n_micro + count > st->cfg.n_micro) return fail(TMPS_ESLOT, "slots %d..%d are not of one mini-batch group", slot, slot + count - 1);
    for (int j = 0; j < count; ++j)
        if (st->slot_used[slot + j]) return fail(TMPS_ESLOT, "slot %d is in use", slot + j);
    if (st->cfg.is_last && !labels) return fail(TMPS_EINVAL, "the last stage needs labels");
    hipStream_t s = (hipStream_t)hip_stream;
    const int mb = st->cfg.micro_batch * count;   // samples of this pass: rows of consecutive slots are consecutive
    const int dt = st->cfg.dtype;
    const int64_t row0 = (int64_t)slot * st->cfg.micro_batch;
    const void* x0 = x;
    if (!st->cfg.borrow_input) {
        char* dst = st->stash + st->in_off + (size_t)row0 * st->in_elems * st->in_esize;
        TMPS_RUN(kcCopy, s, hipMemcpyAsync(dst, x, (size_t)mb * st->in_elems * st->in_esize, hipMemcpyDeviceToDevice, s));
        x0 = dst;
    }
    const size_t x_step = (size_t)st->cfg.micro_batch * st->in_elems * st->in_esize;
    for (int j = 0; j < count; ++j) st->slot_x[slot + j] = (const char*)x + j * x_step;
    if (st->use_graphs && st->cfg.is_last) {
        // a captured loss kernel reads its labels at a fixed address: the stage's own copy of this slot's labels
        int32_t* lab = reinterpret_cast<int32_t*>(st->stash + st->lab_off) + (size_t)row0 * st->label_rps;
        TMPS_RUN(kcCopy, s, hipMemcpyAsync(lab, labels, (size_t)mb * st->label_rps * 4, hipMemcpyDeviceToDevice, s));
        labels = lab;
    }
    const tmps_stage::GraphKey key = {1 + 2 * ((uintptr_t)count + 128 * (uintptr_t)before), (uintptr_t)slot, (uintptr_t)x0, (uintptr_t)labels, (uintptr_t)loss_out, (uintptr_t)ws,
                                      (uintptr_t)st->master, (uintptr_t)st->wcopy};
    // (asked of a whole mini-batch's rows: all of its passes then run the same kernel, however they are cut)
    const bool small_loss = st->cfg.is_last && softmax_ce_small_takes((int64_t)st->M() * st->label_rps, st->layers.back().d.dims[0]);
    float* const y_by_loss = small_loss && !st->use_graphs ? static_cast<float*>(y) : nullptr;
    // The result for the next worker leaves the kernel that forms it in two places, where that is a contraction (a copy afterwards reads it once more: 1.5 MB
    // 3.4 us, 20 MB of logits 8.4, 13 MB 5.1).  Not into what the pass still reads, and not from a captured graph, whose addresses are fixed.
    const size_t out_layer = st->layers.size() - (st->cfg.is_last ? 2 : 1);
    const LayerRT& O = st->layers[out_layer];
    const size_t y_bytes = (size_t)mb * O.out_elems * O.out_esize;
    const bool twice = y && !y_by_loss && !st->use_graphs && (reinterpret_cast<uintptr_t>(y) & 15) == 0 &&
                       !overlap(y, y_bytes, x0, (size_t)mb * st->in_elems * st->in_esize);
    bool y_done = false;
    auto again = [&](size_t li) -> void* {   // for the result of layer li
        if (!twice || li != out_layer) return nullptr;
        y_done = true;
        return y;
    };
    auto skipped = [&](size_t li) -> const void* {   // what a residual connection adds to the result of layer li
        const int src = (int)li - st->layers[li].skip;
        if (!st->layers[li].skip) return nullptr;
        return src == 0 ? x0 : (const void*)st->out_ptr(st->layers[src - 1], row0);
    };
    const int rc = run_or_replay(st, key, s, [&]() -> int {
    for (size_t li = 0; li < st->layers.size(); ++li) {
        const LayerRT& L = st->layers[li];
        void* out = st->out_ptr(L, row0);
        const int32_t* d = L.d.dims;
        const void* in = L.in_t < 0 ? x0 : (const void*)st->out_ptr(st->layers[L.in_t], row0);
        switch (L.d.kind) {
            case TMPS_LINEAR: {
                const void* res = skipped(li);
                void* zout = L.act == 2 ? (void*)(st->stash + L.z_off + (size_t)row0 * L.out_elems * st->asz) : again(li);
                TMPS_GEMM(dense_forward(dt, in, st->wptr(L), st->bptr(L), out, mb * L.rps, d[0], d[1], L.act, L.out_f32, res,
                                        zout, ws, s));
                break;
            }
            case TMPS_CONV2D: {
                // A convolution without activation whose only reader is an affine layer over its channels runs fused with
                // it, and with the residual join after the affine layer when that follows directly.
                const size_t nl = st->layers.size();
                if (L.act == 0 && li + 1 < nl && affine_of_conv(*st, (int)li + 1) && st->readers[li + 1] == 1) {
                    const LayerRT& A = st->layers[li + 1];
                    const bool join = !A.relu && li + 2 < nl && st->layers[li + 2].d.kind == TMPS_RESADD &&
                                      st->readers[li + 2] == 1;
                    if (join) {
                        const LayerRT& J = st->layers[li + 2];
                        const void* b = J.in_b < 0 ? x0 : (const void*)st->out_ptr(st->layers[J.in_b], row0);
                        // the next block's first convolution, which reads the join as a map of its channels, in the same launch
                        if (dt == kBF16 && li + 4 < nl && pointwise_below(*st, (int)li + 1) && pointwise_below(*st, (int)li + 4) && st->layers[li + 3].in_t == (int)li + 2 &&
                            st->layers[li + 3].act == 0 && st->readers[li + 4] == 1 && st->layers[li + 3].d.dims[2] == d[3] && st->layers[li + 3].d.dims[3] == d[2] && li + 4 != out_layer &&
                            pointwise_forward_takes((int64_t)mb * d[0] * d[1], d[2], d[3], true)) {
                            const LayerRT &C = st->layers[li + 3], &B = st->layers[li + 4];
                            const PointwiseForward f{in, st->wptr(L), b, st->bptr(L), st->master + A.w_off, st->master + A.b_off, out, st->out_ptr(J, row0), nullptr, J.relu};
                            const PointwiseForward n{nullptr, st->wptr(C), nullptr, st->bptr(C), st->master + B.w_off, st->master + B.b_off, st->out_ptr(C, row0),
                                                     st->out_ptr(B, row0), nullptr, B.relu};
                            if (on16({f.x, f.w, f.res, f.gain, f.shift, f.z, f.y, n.w, n.z, n.y})) {
                                TMPS_GEMM(pointwise_forward(f, &n, (int64_t)mb * d[0] * d[1], d[2], d[3], s));
                                li += 4;
                                break;
                            }
                        }
                        TMPS_GEMM(conv_affine_forward(dt, in, st->wptr(L), st->bptr(L), out, st->master + A.w_off, st->master + A.b_off,
                                                      again(li + 2), b, st->out_ptr(J, row0), J.relu, conv_shape(L.d, mb), ws, s));
                        li += 2;
                    } else {
                        TMPS_GEMM(conv_affine_forward(dt, in, st->wptr(L), st->bptr(L), out, st->master + A.w_off, st->master + A.b_off,
                                                      again(li + 1), nullptr, st->out_ptr(A, row0), A.relu, conv_shape(L.d, mb), ws, s));
                        li += 1;
                    }
                    break;
                }
                TMPS_GEMM(conv_forward(dt, in, st->wptr(L), st->bptr(L), out, conv_shape(L.d, mb), L.relu, ws, s));
                break;
            }
            case TMPS_MAXPOOL:
                TMPS_GEMM(maxpool_forward(dt, in, out, winners(st, L, row0), mb, d[0], d[1], d[2], d[3], d[4], d[5], s));
                break;
            case TMPS_AFFINE:
                TMPS_GEMM(affine_forward(dt, in, st->master + L.w_off, st->master + L.b_off, out, (int64_t)mb * d[0] * d[1], d[2],
                                         L.relu, s));
                break;
            case TMPS_RESADD: {
                const void* b = L.in_b < 0 ? x0 : (const void*)st->out_ptr(st->layers[L.in_b], row0);
                TMPS_GEMM(resadd_forward(dt, in, b, out, (int64_t)mb * L.out_elems, L.relu, s));
                break;
            }
            case TMPS_AVGPOOL:
                TMPS_GEMM(avgpool_forward(dt, in, out, mb, d[0] * d[1], d[2], s));
                break;
            case TMPS_LAYERNORM: {
                float* stats = reinterpret_cast<float*>(st->stash + L.aux_off) + (size_t)row0 * L.rps * 2;
                if (li + 1 < st->layers.size() && st->layers[li + 1].d.kind == TMPS_LINEAR && st->layers[li + 1].rps == L.rps &&
                    norm_dense_takes(dt, (int64_t)mb * L.rps, d[0], st->layers[li + 1].d.dims[1])) {
                    const LayerRT& F = st->layers[++li];
                    void* zout = F.act == 2 ? (void*)(st->stash + F.z_off + (size_t)row0 * F.out_elems * st->asz) : again(li);
                    TMPS_GEMM(norm_dense_forward(dt, in, st->master + L.w_off, st->master + L.b_off, out, stats, 1e-5f, st->wptr(F), st->bptr(F),
                                                 st->out_ptr(F, row0), mb * L.rps, d[0], F.d.dims[1], F.act, F.out_f32, skipped(li), zout, s));
                    break;
                }
                TMPS_GEMM(layernorm_forward(dt, in, st->master + L.w_off, st->master + L.b_off, out, stats, (int64_t)mb * L.rps, d[0], 1e-5f, s));
                break;
            }
            case TMPS_ATTENTION:
                TMPS_GEMM(attention_forward(dt, in, out,
                                            reinterpret_cast<float*>(st->stash + L.aux_off) + (size_t)row0 * d[2] * d[0], mb,
                                            d[0], d[1], d[2], s));
                break;
            case TMPS_EMBEDDING:
                TMPS_GEMM(embedding_forward(dt, (const int32_t*)in, st->wptr(L), st->bptr_c(L), out, (int64_t)mb * d[1], d[1],
                                            d[2], d[0], s));
                break;
            case TMPS_SOFTMAX_CE: {
                const int rows = mb * L.rps, rows_before = before * st->cfg.micro_batch * L.rps, all = rows_before + rows;
                float* rl = stage_row_loss(st, slot - before);   // (of the rows before, then this pass's)
                if (small_loss) {
                    TMPS_RUN(kcSoftmaxCE, s, softmax_ce_small(dt, (const float*)in, labels, out, y_by_loss, rl, rows, d[0], rows_before,
                                                              1.0f / ((float)st->M() * (float)L.rps), 1.0f / (float)all, loss_out, s));
                    break;
                }
                TMPS_RUN(kcSoftmaxCE, s, softmax_ce(dt, (const float*)in, labels, out, rl + rows_before, rows, d[0],
                                                    1.0f / ((float)st->M() * (float)L.rps), s));
                if (loss_out) TMPS_RUN(kcReduce, s, reduce_scaled_sum(rl, all, 1.0f / (float)all, loss_out, s));
                break;
            }
        }
    }
    return TMPS_OK;
    });
    if (rc != TMPS_OK) return rc;
    if (y && !y_by_loss && !y_done) TMPS_RUN(kcCopy, s, hipMemcpyAsync(y, st->out_ptr(O, row0), y_bytes, hipMemcpyDeviceToDevice, s));
    for (int j = 0; j < count; ++j) st->slot_used[slot + j] = 1;
    return TMPS_OK;
}

extern "C" int tmps_backward(tmps_stage* st, const int* slots, int n_slots, const void* dy, void* dx,
                             void* hip_stream) {
    return backward_between(st, slots, n_slots, dy, dx, hip_stream, 0);
}

bool tmps::can_mask_dx(const tmps_stage& st) {
    bool reads = false;
    for (const LayerRT& L : st.layers) {
        const bool first = L.in_t < 0, joins = L.d.kind == TMPS_RESADD && L.in_b < 0;
        if (joins || (first && L.d.kind != TMPS_LINEAR && L.d.kind != TMPS_CONV2D)) return false;
        reads = reads || first;
        // (a residual connection from the stage input starts at a layer normalisation, which is no such reader)
    }
    return reads;
}

int tmps::backward_between(tmps_stage* st, const int* slots, int n_slots, const void* dy, void* dx, void* hip_stream, int flags) {
    if (!st || !slots) return fail(TMPS_EINVAL, "stage or slots is null");
    const int N = st->cfg.n_micro, mb = st->cfg.micro_batch, M = st->M();
    if (n_slots != N)
        return fail(TMPS_ESLOT, "a backward pass covers the %d micro-batches of one mini-batch, got %d slots", N, n_slots);
    const int g0 = slots[0];
    if (g0 < 0 || g0 % N != 0 || g0 + N > st->cfg.max_stash)
        return fail(TMPS_ESLOT, "slots must be one group g*N..g*N+N-1; first slot is %d", g0);
    for (int j = 0; j < N; ++j) {
        if (slots[j] != g0 + j) return fail(TMPS_ESLOT, "slots of a group must be consecutive");
        if (!st->slot_used[g0 + j]) return fail(TMPS_ESLOT, "slot %d has not been forwarded", g0 + j);
    }
    if (!st->cfg.is_last && !dy) return fail(TMPS_EINVAL, "dy is null on a stage that is not the last");
    hipStream_t s = (hipStream_t)hip_stream;
    const int dt = st->cfg.dtype;
    const int64_t row0 = (int64_t)g0 * mb;

    const char* x0;
    if (st->cfg.borrow_input) {
        x0 = (const char*)st->slot_x[g0];
        const size_t step = (size_t)mb * st->in_elems * st->in_esize;
        for (int j = 1; j < N; ++j)
            if ((const char*)st->slot_x[g0 + j] != x0 + j * step)
                return fail(TMPS_ESHAPE, "borrowed inputs of a mini-batch must be consecutive in memory: slot %d holds %p, expected %p (slot %d + %d x %zu bytes)",
                            g0 + j, st->slot_x[g0 + j], (const void*)(x0 + j * step), g0, j, step);
    } else {
        x0 = st->stash + st->in_off + (size_t)row0 * st->in_elems * st->in_esize;
    }
    // The arguments are accepted.  From here on the slots are given up whatever happens: a pass that fails midway
    // has written part of the gradients, and the stage must be able to take the next mini-batch.
    struct FreeSlots {
        tmps_stage* st; int g0, N;
        ~FreeSlots() {
            for (int j = 0; j < N; ++j) {
                st->slot_used[g0 + j] = 0;
                st->slot_x[g0 + j] = nullptr;
            }
        }
    } free_slots{st, g0, N};

    const tmps_stage::GraphKey key = {2, (uintptr_t)g0, (uintptr_t)x0, (uintptr_t)dy, (uintptr_t)dx, (uintptr_t)flags,
                                      (uintptr_t)st->master, (uintptr_t)st->wcopy};
    return run_or_replay(st, key, s, [&]() -> int {
    // Gradients are kept per result: grads[t + 1] is the gradient w.r.t. the result of layer t (t = -1: the stage
    // input).  Layers are visited last to first; every layer that reads a result contributes to its gradient: the
    // first contribution is written, later ones are added to what is there (in the epilogue of the kernel that
    // computes them).  Buffers come from a small pool and are shared by reference count: a residual connection
    // hands the SAME gradient to both of its sources without copying it.
    struct Grad {
        const void* ptr = nullptr;
        int buf = -1;      // pool buffer that holds it; -1: memory that is not ours to write or free (dy, the stash, dx)
        bool set = false;
        bool masked = false;   // it has passed through the activation of the layer whose result it belongs to
    };
    const int nl = (int)st->layers.size();
    std::vector<Grad> grads(nl + 1);
    std::vector<int> remaining(st->readers);
    char* gbuf[8];
    int refs[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int k = 0; k < st->n_gbuf; ++k) gbuf[k] = st->scratch + st->gbuf_off[k];
    auto take = [&]() -> int {
        for (int k = 0; k < st->n_gbuf; ++k)
            if (refs[k] == 0) {
                refs[k] = 1;
                return k;
            }
        return -1;
    };
    auto release = [&](int buf) {
        if (buf >= 0) --refs[buf];
    };
    float* ws = reinterpret_cast<float*>(st->scratch + st->ws_off);
    // the stored activation that a gradient written for result t has to pass through (mode 1: ReLU, 2: GELU)
    auto mask_of = [&](int t, int& mode) -> const void* {
        mode = 1;
        if (t < 0) return (flags & kMaskDx) ? (const void*)x0 : nullptr;   // (the stage input is that activation's result)
        const LayerRT& P = st->layers[t];
        if (P.act == 1) return st->out_ptr(P, row0);
        if (P.act == 2) {
            mode = 2;
            return st->stash + P.z_off + (size_t)row0 * P.out_elems * st->asz;
        }
        return nullptr;
    };
    // Where the contribution of a kernel to result t goes: `dst` to write, `add` to join first (null: nothing yet).
    struct Target {
        void* dst = nullptr;
        const void* add = nullptr;
        int buf = -1;
        bool wanted = false;
    };
    auto target = [&](int t, Target& T) -> int {
        T = Target();
        Grad& G = grads[t + 1];
        if (t < 0) {
            if (!dx) return TMPS_OK;   // nobody wants the gradient w.r.t. the stage input
            T.wanted = true;
            T.dst = dx;
            T.add = G.set ? G.ptr : nullptr;
            return TMPS_OK;
        }
        T.wanted = true;
        if (st->layers[t].keep_off) {   // memory of its own
            T.dst = st->scratch + st->layers[t].keep_off;
            T.add = G.set ? G.ptr : nullptr;
            return TMPS_OK;
        }
        if (G.set && G.buf >= 0 && refs[G.buf] == 1) {   // ours alone: add in place
            T.dst = gbuf[G.buf];
            T.add = G.ptr;
            T.buf = G.buf;
            return TMPS_OK;
        }
        T.buf = take();
        if (T.buf < 0 && dx && grads[0].set && grads[0].buf >= 0) {   // (what dx is still to be added to holds one)
            TMPS_RUN(kcCopy, s, copy_bytes(dx, grads[0].ptr, (size_t)M * st->in_elems * st->asz, s));
            release(grads[0].buf);
            grads[0].ptr = dx;
            grads[0].buf = -1;
            T.buf = take();
        }
        if (T.buf < 0) return fail(TMPS_EUNSUPPORTED, "out of gradient buffers (too many open residual connections)");
        T.dst = gbuf[T.buf];
        T.add = G.set ? G.ptr : nullptr;
        return TMPS_OK;
    };
    auto commit = [&](int t, const Target& T) {
        Grad& G = grads[t + 1];
        if (G.set && G.buf != T.buf) release(G.buf);
        G.ptr = T.dst;
        G.buf = T.buf;
        G.set = true;
        G.masked = true;   // (by the kernel that wrote it)
        --remaining[t + 1];
    };
    // A caller may have the gradient w.r.t. the input written over the upstream gradient or the input: then every kernel that reads
    // those comes, as they are called, before the one that writes.
    const size_t dx_bytes = (size_t)M * st->in_elems * st->asz;
    const bool in_order = overlap(dx, dx_bytes, dy, (size_t)M * st->out_elems * st->asz) || overlap(dx, dx_bytes, x0, (size_t)M * st->in_elems * st->in_esize);
    // hand an existing gradient (g) to result t as its contribution, without a kernel when it is the first
    auto share = [&](int t, const Grad& g) -> int {
        if (t < 0 && !dx) return TMPS_OK;
        Grad& G = grads[t + 1];
        const int64_t n = (int64_t)M * st->tensor_elems(t);
        if (t < 0 && (G.set || in_order || remaining[0] == 1)) {
            if (G.set) TMPS_GEMM(resadd_forward(dt, G.ptr, g.ptr, dx, n, 0, s));
            else TMPS_RUN(kcCopy, s, copy_bytes(dx, g.ptr, (size_t)n * st->asz, s));
            release(G.buf);
            G.ptr = dx; G.buf = -1; G.set = true;
        } else if (!G.set) {
            // (also of the stage input: the layer that reads it beside this one adds this to its own contribution and writes dx)
            G = g;
            if (g.buf >= 0) ++refs[g.buf];
        } else {
            Target T;
            int rc = target(t, T);
            if (rc != TMPS_OK) return rc;
            TMPS_GEMM(resadd_forward(dt, T.add, g.ptr, T.dst, n, 0, s));
            if (G.buf != T.buf) release(G.buf);
            G.ptr = T.dst; G.buf = T.buf;
        }
        G.masked = false;
        --remaining[t + 1];
        return TMPS_OK;
    };

    Reductions sums;   // left to the end of the pass
    auto partials = [&](const LayerRT& L) {
        return L.part_elems ? Partials(reinterpret_cast<float*>(st->scratch + L.part_off), &sums) : Partials(ws);
    };
    std::vector<DenseWgradJob> waiting;
    int waiting_rows = 0;
    auto flush_group = [&]() -> int {
        if (waiting.empty()) return TMPS_OK;
        TMPS_GEMM(dense_wgrad_group(dt, waiting.data(), (int)waiting.size(), waiting_rows, ws, (int64_t)(st->ws_bytes / 4), s));
        waiting.clear();
        return TMPS_OK;
    };

    // The input gradient of a 1 x 1 convolution with a stride touches few positions of its input's gradient.  Where other layers read the same input
    // it comes last, added in place, instead of first over the whole map (one at a time: its own gradient is kept until then).
    struct {
        int li = -1;
        Grad g;
    } strided;
    auto conv_input_gradient = [&](int li, const Grad& g) -> int {
        const LayerRT& L = st->layers[li];
        ConvShape c = conv_shape(L.d, M);
        int mode;
        const void* mask = mask_of(L.in_t, mode);
        Target T;
        int rc = target(L.in_t, T);
        if (rc != TMPS_OK || !T.wanted) return rc;
        if (mode == 2) return fail(TMPS_EUNSUPPORTED, "a convolution directly after a GELU layer");
        c.rest_done = T.add && T.add == T.dst && (!mask || grads[L.in_t + 1].masked);
        TMPS_GEMM(conv_dgrad(dt, g.ptr, st->wptr(L), T.dst, mask, T.add, c, ws, s));
        commit(L.in_t, T);
        return TMPS_OK;
    };
    auto can_wait = [&](const LayerRT& L) {
        const int32_t* d = L.d.dims;
        return strided.li < 0 && !in_order && d[4] == 1 && d[5] == 1 && d[6] > 1 && d[7] == 0 && remaining[L.in_t + 1] > 1 && !grads[L.in_t + 1].set &&
               (L.in_t >= 0 || dx) && std::count(refs, refs + st->n_gbuf, 0) >= 3;
    };
    auto strided_is_last = [&]() { return strided.li >= 0 && remaining[st->layers[strided.li].in_t + 1] == 1; };

    int top = nl - 1;
    if (st->cfg.is_last) {
        // the loss layer's contribution to the logits: the softmax error signal stored by the forward passes
        Grad& G = grads[top];   // result top - 1
        G.ptr = st->out_ptr(st->layers[top], row0);
        G.buf = -1;
        G.set = true;
        --remaining[top];
        --top;
    } else {
        Grad& G = grads[top + 1];
        G.ptr = dy;
        G.buf = -1;
        G.set = true;
        const LayerRT& T = st->layers[top];
        if (T.relu && !(flags & kDyMasked)) {
            const int k = take();
            TMPS_RUN(kcReluMask, s, relu_mask(dt, dy, st->out_ptr(T, row0), gbuf[k], (int64_t)M * T.out_elems, s));
            G.ptr = gbuf[k];
            G.buf = k;
        }
    }
    for (int li = top; li >= 0; --li) {
        const LayerRT& L = st->layers[li];
        const int32_t* d = L.d.dims;
        const Grad g = grads[li + 1];
        if (!g.set || remaining[li + 1] != 0) return fail(TMPS_ESHAPE, "layer %d: its result has no complete gradient", li);
        const int t_in = L.in_t;
        const void* in = t_in < 0 ? (const void*)x0 : (const void*)st->out_ptr(st->layers[t_in], row0);
        int mask_mode = 1;
        const void* mask = mask_of(t_in, mask_mode);
        float* gw = st->grad + L.w_off;
        Target T;
        int rc, with_below = 0;   // layers below whose backward pass this one's includes
        switch (L.d.kind) {
            case TMPS_LINEAR: {
                const int rows = M * L.rps;
                if (L.skip && (rc = share(st->layers[li - L.skip].in_t, g)) != TMPS_OK) return rc;
                if ((rc = target(t_in, T)) != TMPS_OK) return rc;
                // (the gradient in a buffer that is about to be used again, or an operand that a user has put at an odd address: at once)
                const bool later = L.grouped && !in_order && g.buf < 0 && ((reinterpret_cast<uintptr_t>(g.ptr) | reinterpret_cast<uintptr_t>(in)) & 15) == 0;
                if (later) {
                    if (waiting_rows != rows || (int)waiting.size() == kWgradGroupMax) {
                        if ((rc = flush_group()) != TMPS_OK) return rc;
                    }
                    waiting_rows = rows;
                    waiting.push_back(DenseWgradJob{g.ptr, in, gw, d[0], d[1]});
                    if (T.wanted) TMPS_GEMM(dense_dgrad(dt, g.ptr, st->wptr(L), T.dst, mask, mask_mode, T.add, rows, d[0], d[1], ws, s));
                } else if (T.wanted && !in_order) {
                    TMPS_GEMM(dense_backward(dt, g.ptr, in, st->wptr(L), gw, T.dst, mask, mask_mode, T.add, rows, d[0], d[1], ws, partials(L), s));
                } else {
                    TMPS_GEMM(dense_wgrad(dt, g.ptr, in, gw, rows, d[0], d[1], partials(L), s));
                    if (T.wanted) TMPS_GEMM(dense_dgrad(dt, g.ptr, st->wptr(L), T.dst, mask, mask_mode, T.add, rows, d[0], d[1], ws, s));
                }
                if (T.wanted) commit(t_in, T);
                break;
            }
            case TMPS_CONV2D: {
                TMPS_GEMM(conv_wgrad(dt, g.ptr, in, gw, conv_shape(L.d, M), partials(L), s));
                if (can_wait(L)) {
                    strided.li = li;
                    strided.g = g;
                    if (g.buf >= 0) ++refs[g.buf];
                } else if ((rc = conv_input_gradient(li, g)) != TMPS_OK) return rc;
                break;
            }
            case TMPS_MAXPOOL: {
                const void* won = winners(st, L, row0);
                const LayerRT* A = t_in >= 0 && st->layers[t_in].d.kind == TMPS_AFFINE && st->layers[t_in].d.dims[2] == d[2] ? &st->layers[t_in] : nullptr;
                const int64_t rows = (int64_t)M * d[0] * d[1];
                if (A && st->readers[t_in + 1] == 1 && !in_order && maxpool_affine_takes(dt, rows, d[2], d[3], d[4])) {
                    if ((rc = target(A->in_t, T)) != TMPS_OK) return rc;
                    if (T.add) return fail(TMPS_EUNSUPPORTED, "an affine layer on a shared input");
                    const void* const z = A->in_t < 0 ? (const void*)x0 : (const void*)st->out_ptr(st->layers[A->in_t], row0);
                    if (T.wanted && ((reinterpret_cast<uintptr_t>(g.ptr) | reinterpret_cast<uintptr_t>(z) | reinterpret_cast<uintptr_t>(T.dst)) & 15) == 0) {
                        TMPS_GEMM(maxpool_affine_backward(dt, g.ptr, won, z, st->master + A->w_off, T.dst, st->grad + A->w_off, partials(*A), M, d[0], d[1], d[2], d[3],
                                                          d[4], d[5], mask ? 1 : 0, s));
                        commit(A->in_t, T);
                        --remaining[t_in + 1];
                        with_below = 1;
                        break;
                    }
                    release(T.buf);
                }
                if ((rc = target(t_in, T)) != TMPS_OK) return rc;
                if (T.wanted) {
                    if (T.add || mask_mode == 2) return fail(TMPS_EUNSUPPORTED, "max pooling on a shared or GELU input");
                    TMPS_GEMM(maxpool_backward(dt, g.ptr, won, T.dst, M, d[0], d[1], d[2], d[3], d[4], d[5], mask ? 1 : 0, s));
                    commit(t_in, T);
                }
                break;
            }
            case TMPS_AVGPOOL:
                if ((rc = target(t_in, T)) != TMPS_OK) return rc;
                if (T.wanted) {
                    if (T.add || mask_mode == 2) return fail(TMPS_EUNSUPPORTED, "average pooling on a shared or GELU input");
                    TMPS_GEMM(avgpool_backward(dt, g.ptr, in, T.dst, M, d[0] * d[1], d[2], mask ? 1 : 0, s));
                    commit(t_in, T);
                }
                break;
            case TMPS_AFFINE:
                // the layer before has no activation (checked at creation): nothing to pass through
                if (pointwise_below(*st, li) && st->readers[t_in + 1] == 1 && !in_order) {
                    const LayerRT& C = st->layers[li - 1];
                    const int64_t P = (int64_t)M * d[0] * d[1];
                    const int I = C.d.dims[2];
                    const void* const x = C.in_t < 0 ? (const void*)x0 : (const void*)st->out_ptr(st->layers[C.in_t], row0);
                    const Grad& G = grads[C.in_t + 1];
                    int mode;
                    const void* const relu = mask_of(C.in_t, mode);
                    if (affine_pointwise_takes(dt, P, d[2], I) && L.part_elems && C.part_elems && mode == 1 && (C.in_t >= 0 || dx) &&
                        on16({g.ptr, in, x, st->master + L.w_off, G.set ? G.ptr : nullptr, C.in_t < 0 ? dx : nullptr})) {
                        if ((rc = target(C.in_t, T)) != TMPS_OK) return rc;
                        TMPS_GEMM(affine_pointwise_backward(g.ptr, in, x, st->wptr(C), st->master + L.w_off, T.add, relu ? 1 : 0, T.dst, gw, st->grad + C.w_off,
                                                            partials(L), partials(C), P, d[2], I, s));
                        commit(C.in_t, T);
                        --remaining[t_in + 1];
                        with_below = 1;
                        break;
                    }
                }
                if ((rc = target(t_in, T)) != TMPS_OK) return rc;
                if (T.add) return fail(TMPS_EUNSUPPORTED, "an affine layer on a shared input");
                TMPS_GEMM(affine_backward(dt, g.ptr, in, st->master + L.w_off, T.wanted ? T.dst : nullptr, gw, partials(L),
                                          (int64_t)M * d[0] * d[1], d[2], s));
                if (T.wanted) commit(t_in, T);
                break;
            case TMPS_RESADD:
                // d(a + b) = the incoming gradient for both sources (it has already passed through this layer's ReLU)
                if ((rc = share(L.in_b, g)) != TMPS_OK) return rc;
                if ((rc = share(t_in, g)) != TMPS_OK) return rc;
                break;
            case TMPS_LAYERNORM:
                if (mask) return fail(TMPS_EUNSUPPORTED, "layer normalisation directly after an activation");
                if ((rc = target(t_in, T)) != TMPS_OK) return rc;
                TMPS_GEMM(layernorm_backward(dt, g.ptr, in, reinterpret_cast<const float*>(st->stash + L.aux_off) + (size_t)row0 * L.rps * 2,
                                             st->master + L.w_off, T.add, T.wanted ? T.dst : nullptr, gw, partials(L), (int64_t)M * L.rps,
                                             d[0], s));
                if (T.wanted) commit(t_in, T);
                break;
            case TMPS_ATTENTION:
                if (mask) return fail(TMPS_EUNSUPPORTED, "attention directly after an activation");
                if ((rc = target(t_in, T)) != TMPS_OK) return rc;
                if (T.wanted) {
                    if (T.add) return fail(TMPS_EUNSUPPORTED, "attention on a shared input");
                    TMPS_GEMM(attention_backward(dt, in, st->out_ptr(L, row0), g.ptr,
                                                 reinterpret_cast<const float*>(st->stash + L.aux_off) + (size_t)row0 * d[2] * d[0], ws,
                                                 T.dst, M, d[0], d[1], d[2], s));
                    commit(t_in, T);
                }
                break;
            case TMPS_EMBEDDING:
                TMPS_GEMM(embedding_backward(dt, (const int32_t*)in, g.ptr, gw, st->grad + L.b_off, M, d[1], d[2], d[0], s));
                break;
            default:
                return fail(TMPS_EUNSUPPORTED, "layer kind %d has no backward", L.d.kind);
        }
        release(g.buf);
        grads[li + 1].set = false;
        if (strided_is_last()) {
            if ((rc = conv_input_gradient(strided.li, strided.g)) != TMPS_OK) return rc;
            release(strided.g.buf);
            strided.li = -1;
        }
        // A result whose gradient is complete but was only handed over (never written through a kernel that applies
        // the activation of its producer) still has to pass through that activation.
        if (t_in >= 0 && remaining[t_in + 1] == 0 && grads[t_in + 1].set && L.d.kind == TMPS_RESADD) {
            int mm = 1;
            const void* mk = mask_of(t_in, mm);
            if (mk) return fail(TMPS_EUNSUPPORTED, "a residual join whose first source ends in an activation");
        }
        if (L.d.kind == TMPS_RESADD && L.in_b >= 0 && remaining[L.in_b + 1] == 0 && st->layers[L.in_b].act != 0)
            return fail(TMPS_EUNSUPPORTED, "a residual connection must start at a result that another, earlier layer reads too");
        li -= with_below;
    }
    int rc = flush_group();
    if (rc != TMPS_OK) return rc;
    TMPS_GEMM(reduce_all(sums, s));
    return TMPS_OK;
    });   // (free_slots releases the group)
}

// What a pair of timing events costs by itself on this stream: the brackets of its launches hold one each.
static void empty_bracket(hipStream_t s) { ProfileScope empty(kcEventPair, s); }

extern "C" int tmps_update(tmps_stage* st, void* hip_stream) {
    if (!st) return fail(TMPS_EINVAL, "stage is null");
    hipStream_t s = (hipStream_t)hip_stream;
    empty_bracket(s);
    if (st->shadow_n > 0) {
        // the version about to be superseded is kept for the passes tagged with it: the update stores what it replaces
        const int slot = (int)(st->version % st->shadow_n);
        float* const kept = reinterpret_cast<float*>(st->shadow + (size_t)slot * st->param_bytes);
        TMPS_RUN(kcUpdate, s, sgd_momentum_keeping(st->master, st->mom, st->grad, st->wcopy, st->P, st->cfg.lr, st->cfg.momentum, kept,
                                                   st->wcopy ? (void*)(kept + st->P) : nullptr, s));
        st->shadow_ver[slot] = st->version;
    } else {
        TMPS_RUN(kcUpdate, s, sgd_momentum(st->master, st->mom, st->grad, st->wcopy, st->P, st->cfg.lr, st->cfg.momentum, s));
    }
    ++st->version;
    return TMPS_OK;
}

int tmps::update_all(tmps_stage* const* stages, int n, void* hip_stream) {
    hipStream_t s = (hipStream_t)hip_stream;
    Update list[kUpdateMax];
    int k = 0;
    auto flush = [&]() -> int {
        if (k == 0) return TMPS_OK;
        empty_bracket(s);
        TMPS_RUN(kcUpdate, s, sgd_momentum_all(list, k, s));
        k = 0;
        return TMPS_OK;
    };
    int rc;
    for (int i = 0; i < n; ++i) {
        tmps_stage* st = stages[i];
        if (n == 1 || st->shadow_n > 0) {
            if ((rc = tmps_update(st, hip_stream)) != TMPS_OK) return rc;
            continue;
        }
        if (k == kUpdateMax && (rc = flush()) != TMPS_OK) return rc;
        list[k++] = Update{st->master, st->mom, st->grad, st->wcopy, st->P, st->cfg.lr, st->cfg.momentum};
        ++st->version;
    }
    return flush();
}

extern "C" int tmps_backward_at(tmps_stage* st, long version, const int* slots, int n_slots, const void* dy, void* dx,
                                void* hip_stream) {
    return backward_between_at(st, version, slots, n_slots, dy, dx, hip_stream, 0);
}

int tmps::backward_between_at(tmps_stage* st, long version, const int* slots, int n_slots, const void* dy, void* dx, void* hip_stream, int flags) {
    if (!st) return fail(TMPS_EINVAL, "stage is null");
    if (version == st->version) return backward_between(st, slots, n_slots, dy, dx, hip_stream, flags);
    int found = -1;
    for (int k = 0; k < st->shadow_n; ++k)
        if (st->shadow_ver[k] == version) found = k;
    if (found < 0)
        return fail(TMPS_EINVAL, "weights after %ld updates are not kept (the stage is at %ld and keeps %d older versions)",
                    version, st->version, st->shadow_n);
    // as in tmps_forward_micro_at: the kernels take their weight pointers at launch; the gradients still go to the
    // stage's own gradient array, and the update that follows changes the live weights
    float* const live_master = st->master;
    void* const live_wcopy = st->wcopy;
    char* base = st->shadow + (size_t)found * st->param_bytes;
    st->master = reinterpret_cast<float*>(base);
    if (live_wcopy) st->wcopy = base + (size_t)st->P * 4;
    const int rc = backward_between(st, slots, n_slots, dy, dx, hip_stream, flags);
    st->master = live_master;
    st->wcopy = live_wcopy;
    return rc;
}

int tmps::forward_run_at(tmps_stage* st, long version, int slot, int count, const void* x, void* y, const int32_t* labels,
                         float* loss_out, void* hip_stream, int before) {
    float* const ws = reinterpret_cast<float*>(st->scratch + st->ws_off);
    if (version == st->version) return forward_with_workspace(st, slot, count, x, y, labels, loss_out, hip_stream, ws, before);
    int found = -1;
    for (int k = 0; k < st->shadow_n; ++k)
        if (st->shadow_ver[k] == version) found = k;
    if (found < 0)
        return fail(TMPS_EINVAL, "weights after %ld updates are not kept (the stage is at %ld and keeps %d older versions)",
                    version, st->version, st->shadow_n);
    // The kernels take their weight pointers when they are launched: point the stage at the kept copy for the
    // duration of this call.  (Calls on one stage come from one host thread at a time.)
    float* const live_master = st->master;
    void* const live_wcopy = st->wcopy;
    char* base = st->shadow + (size_t)found * st->param_bytes;
    st->master = reinterpret_cast<float*>(base);
    if (live_wcopy) st->wcopy = base + (size_t)st->P * 4;
    const int rc = forward_with_workspace(st, slot, count, x, y, labels, loss_out, hip_stream, ws, before);
    st->master = live_master;
    st->wcopy = live_wcopy;
    return rc;
}

extern "C" int tmps_forward_micro_at(tmps_stage* st, long version, int slot, const void* x, void* y, const int32_t* labels,
                                     float* loss_out, void* hip_stream) {
    if (!st) return fail(TMPS_EINVAL, "stage is null");
    return forward_run_at(st, version, slot, 1, x, y, labels, loss_out, hip_stream, 0);
}
