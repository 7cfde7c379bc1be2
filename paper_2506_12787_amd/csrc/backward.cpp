// Backward pass orchestration (blend -> preprocess -> MLP) and its C ABI entry.
#include <algorithm>

#include "runtime.h"

namespace swf {

// MLP backward, every GEMM in this library's own kernels. The hidden
// activations are the ones the forward's MLP kernel stored (the values the
// forward used: FP32, or BF16 after a BF16 forward). From dy (gradients of the
// 7 residuals per pair):
//   dW_l = dz_l^T act_{l-1}, db_l = colsum(dz_l), dz_{l-1} = (dz_l W_l) * [act_{l-1} > 0],
// and for layer 1 the weight gradient splits into the mean part
// (sum over queries of dz_0 per Gaussian = S)^T gamma(mu_hat) and the TX part
// (sum over Gaussians of dz_0 per query)^T gamma(s_hat); the mean features'
// gradient is S W1m, taken through the sin / cos features to d mu.
// bf16: the backward of a BF16 forward. dz is stored in BF16 (FP32 sums, then
// one rounding) and the 256 x 256 products run on BF16 matrix cores with FP32
// accumulation; FP32: the products run on the FP32 matrix cores.
// Weight and bias gradients are accumulated in FP32 either way.
// Only the rows of rg (pairs with a gradient, in groups of 32) are taken: a row whose dy is zero has zero dz in every
// layer.
swf_status Ctx::mlp_backward(Workspace& w, const DevScene& d, const float* tx, int B, const float* dy,
                             const RowGroups& rg, const swf_grads* gr, bool bf16, hipStream_t st) {
    swf_status s = SWF_OK;
    const int64_t N = d.n, P = (int64_t)B * N;
    const int nh = d.n_hidden, Hd = 256, I = d.in_dim;
    const size_t actb = act_layer_bytes(P, bf16);
    const size_t f32b = (size_t)P * Hd * sizeof(float);
    if (!w.act.ptr || w.act.cap < actb * nh) return fail(SWF_E_STATE, "the forward's activations are missing");
    // dz ping-pong; BF16 with a single hidden layer: also the FP32 layer-1 gradient (formed inside its sums)
    const bool need_zf = bf16 && nh == 1;
    if ((s = w.dz.reserve(this, need_zf ? actb * 2 + f32b + 16 : actb * 2 + 16, st))) return s;
    // scratch: S (N x 256), R (B x 256), the launches' slices, column-sum partials, packed weights. Only what this
    // backward's launches take: the layer-1 slices of the form it runs, the column sums where those are many, BF16 dy
    // where it is multiplied (500k Gaussians x 64 queries, BF16, four hidden layers: 0.78 GB, 2.11 with all of them)
    const int rblocks = bf16 && nh > 1 ? layer1_grad_blocks((int)N) : layer1_sums_blocks((int)N);
    const size_t n_split = std::max({mean_grad_floats(N), gemm_part_floats(Hd, kTxFeat, B, false),
                                     (size_t)rblocks * B * Hd, out_bwd_floats(P),
                                     bf16 ? wgrad_mfma_floats(P) : wgrad_f32_floats(P)});
    const bool many = rblocks > 512;  // slices of the sums over Gaussians: column sums in two stages
    const size_t n_cs = many ? (size_t)colsum_blocks(rblocks) * Hd * B : 0;
    const size_t n_wb =
        bf16 ? ((size_t)(nh - 1) * Hd * Hd + (size_t)kOut * Hd + (need_zf ? (size_t)P * kOut : 0) + 64) / 2 + 64 : 0;
    const size_t n_wt = bf16 ? 0 : (size_t)(nh - 1) * Hd * Hd;  // FP32: W^T of the 256 x 256 layers, fragment-major
    const size_t small =
        ((size_t)N * Hd + (size_t)B * Hd + 4 + n_split + n_cs + n_wb + n_wt + 64) *
        sizeof(float);
    if ((s = w.part.reserve(this, small, st))) return s;
    if ((s = w.ftx.reserve(this, (size_t)B * kTxFeat * sizeof(float) + 16, st))) return s;
    if ((s = w.dmu.reserve(this, (size_t)N * 2 * sizeof(float) + 16, st))) return s;
    if ((s = w.qs.reserve(this, (size_t)B * Hd * sizeof(float), st))) return s;
    void* act[8] = {};
    for (int l = 0; l < nh; ++l) act[l] = (char*)w.act.ptr + actb * l;
    void* dz[2] = {w.dz.ptr, (char*)w.dz.ptr + actb};
    float* zf = need_zf ? (float*)((char*)w.dz.ptr + actb * 2) : nullptr;  // FP32 layer-1 gradient (nh == 1)
    float* S = (float*)w.part.ptr;               // N x 256
    float* R = S + (size_t)N * Hd;               // B x 256
    float* part = R + (size_t)B * Hd;            // slices (16-byte aligned)
    float* tmp = part + n_split;                 // column-sum partials
    // BF16 weights (launch_pack_bwd), then dy
    uint16_t* wb = (uint16_t*)(((uintptr_t)(tmp + n_cs) + 15) & ~(uintptr_t)15);
    float* wt = (float*)(((uintptr_t)(tmp + n_cs + n_wb) + 15) & ~(uintptr_t)15);  // FP32 W^T, 16-byte aligned
    float *ftx = (float*)w.ftx.ptr, *qs = (float*)w.qs.ptr;
    launch_tx_features(d, tx, B, qs, nullptr, st, ftx);
    uint16_t* wl[8] = {};
    if (bf16) {
        for (int l = 1; l <= nh; ++l) wl[l] = wb + (size_t)(l - 1) * Hd * Hd;
        launch_pack_bwd(d.w, nh, wb, st);
    } else {
        for (int l = 1; l < nh; ++l) launch_pack_wt(d.w[l], wt + (size_t)(l - 1) * Hd * Hd, st);
    }
    // ---- output layer (7 outputs): one pass over the last activations gives its weight and bias gradients and the
    // masked gradient of the last hidden pre-activations (K = 7); BF16 with one hidden layer forms that one below,
    // in FP32 and before its ReLU mask (applied inside the layer-1 sums)
    launch_out_bwd(bf16, dy, bf16 ? (const void*)wl[nh] : d.w[nh], act[nh - 1], P, rg, need_zf ? nullptr : dz[0], part,
                   gr->weight[nh], gr->bias[nh], st);
    if (need_zf) {
        uint16_t* dyb = wl[nh] + (size_t)kOut * Hd;
        launch_to_bf16(dy, P * kOut, dyb, st);
        launch_gemm_f32(false, false, P, Hd, kOut, dyb, kOut, wl[nh], Hd, zf, Hd, part, st, true);
    }
    int cur = 0;
    const void* dz1 = nullptr;  // BF16: the second layer's pre-activation gradient
    for (int l = nh - 1; l >= 1; --l) {
        if (bf16) {
            // contraction over pairs; the bias gradient (column sums of dz) rides along
            launch_wgrad_mfma(dz[cur], act[l - 1], P, rg, part, gr->weight[l], gr->bias[l], st);
            // dz W on MFMA in one pass, BF16 and masked by the previous ReLU; the layer-1 gradient is formed
            // inside its sums below
            if (l > 1)
                launch_dz_gemm(dz[cur], wl[l], act[l - 1], P, rg, dz[cur ^ 1], st);
            else
                dz1 = dz[cur];
        } else {
            launch_wgrad_f32((const float*)dz[cur], (const float*)act[l - 1], P, rg, part, gr->weight[l], gr->bias[l],
                             st);
            // the input gradient on the FP32 matrix cores with the layer's W^T as weights, masked
            launch_dz_f32((const float*)dz[cur], wt + (size_t)(l - 1) * Hd * Hd, (const float*)act[l - 1], P, rg,
                          (float*)dz[cur ^ 1], st);
        }
        cur ^= 1;
    }
    // ---- layer 1: the gradient of its pre-activations dz0, FP32; S = its sum over the batch per Gaussian
    // (N x 256), R = its sum over the Gaussians per query (B x 256), b0 = its sum over all pairs
    if (dz1) {
        // dz0 = (dz1 W1) masked, never stored: one pass gives S and per-block partial sums of R
        launch_layer1_grad(dz1, wl[1], act[0], (int)B, (int)N, rg, S, part, st);
    } else {
        // BF16 with one hidden layer: zf is dz0 before the ReLU mask. FP32: dz0 carries layer 1's ReLU mask already
        // (applied where it was formed). One pass gives S and per-block partial sums of R
        launch_layer1_sums(need_zf ? zf : (const float*)dz[cur], need_zf ? act[0] : nullptr,
                           need_zf ? nullptr : rg.bits, (int)B, (int)N, S, part, st);
    }
    if (gr->weight[0]) {
        if (many)
            launch_colsum(part, rblocks, (int64_t)B * Hd, tmp, R, st);
        else
            launch_slice_sum(part, rblocks, (int64_t)B * Hd, R, st);
    }
    // dW1 [256 x 89] = [S^T gamma(mu_hat) | R^T gamma(s_hat)]; the mean part with b0 (the sum of S over Gaussians) and
    // d mu, through d gamma(mu_hat) = S W1m
    if (gr->weight[0])
        launch_gemm_f32(true, false, Hd, kTxFeat, B, R, Hd, ftx, kTxFeat, gr->weight[0] + kMeanFeat, I, part, st,
                        false);
    launch_mean_grad(S, d, part, gr->weight[0], gr->bias[0], (float*)w.dmu.ptr, st);
    return hip(hipGetLastError(), "mlp backward");
}

swf_status Ctx::backward(Workspace& w, int sid, const float* tx, int B, int flags, const float* grad_out, const void* aux,
                         const swf_grads* gr, hipStream_t st) {
    if (!grad_out || !aux || !gr) return fail(SWF_E_INVALID, "grad_out, aux and grads are required");
    Scene* sc = scene(sid);
    if (!sc) return fail(SWF_E_NOT_FOUND, "unknown scene id");
    if (sc->d.kind == 1) return fail(SWF_E_INVALID, "paper-model scenes have no backward in this library");
    AuxTag t;
    {
        // the forward state used below must be that of the render that filled aux
        auto it = aux_tags.find(aux);
        if (it == aux_tags.end())
            return fail(SWF_E_STATE, "aux was not filled by a swf_render with SWF_KEEP_AUX on this context");
        t = it->second;
        if (t.scene != sid || t.B != B || t.flags != (flags & ~(SWF_KEEP_AUX | SWF_DETERMINISTIC)))
            return fail(SWF_E_INVALID, "scene, batch or flags differ from the render that filled aux");
        if (t.gen != sc->gen)
            return fail(SWF_E_STATE, "the scene's parameters were updated after the render that filled aux");
    }
    const DevScene& d = sc->d;
    const bool deform = !(flags & SWF_NO_DEFORM);
    const bool want_mlp = deform && d.has_mlp;
    // The MLP backward takes the hidden activations the forward's MLP kernel stored (the values the forward
    // used, FP32 or BF16).
    const bool bf16 = (flags & SWF_MLP_BF16) != 0;
    const bool acts_ready = want_mlp && B >= 1 && (uint64_t)B * (uint64_t)d.n < (1ull << 32);
    if (want_mlp && !acts_ready) return fail(SWF_E_INVALID, "the MLP backward takes fewer than 2^32 pairs");
    swf_status s = SWF_OK;
    // 1. the forward's records and lists: still in the workspace if no pass wrote records since that render
    // (and it was given the same positions), else built again (deterministic: identical to the forward's)
    const bool kept = t.seq == w.seq && t.tx == tx && (!acts_ready || t.acts);
    if (!kept) {
        if (acts_ready) {
            const size_t actb = act_layer_bytes((int64_t)B * d.n, bf16);
            if ((s = w.act.reserve(this, actb * d.n_hidden + 16, st))) return s;
            w.act_out = w.act.ptr;
        }
        s = forward_lists(w, sid, tx, B, flags & ~(SWF_KEEP_AUX | SWF_DETERMINISTIC), st);
        w.act_out = nullptr;
        if (s) return s;
    }
    last_bwd_reused = kept;
    const int64_t P = (int64_t)B * d.n;
    const size_t npix = (size_t)B * d.H * d.W;
    const float* auxT = (const float*)aux;
    const uint32_t* auxL = (const uint32_t*)((const char*)aux + sizeof(float) * npix);
    // 2. blend backward -> per-pair gradients of (mean, M, opacity, amp)
    if ((s = w.dpair.reserve(this, (size_t)P * 8 * sizeof(float) + 16, st))) return s;
    if ((s = w.dbase.reserve(this, (size_t)P * kOut * sizeof(float) + 16, st))) return s;
    if ((s = hip(hipMemsetAsync(w.dpair.ptr, 0, (size_t)P * 8 * sizeof(float), st), "memset dpair"))) return s;
    stage_begin(SWF_STAGE_BWD_BLEND, st);
    float* det_part = nullptr;
    const uint32_t* det_off = nullptr;
    if (flags & SWF_DETERMINISTIC) {
        // per (list entry, wave) sums, zero where a wave contributes nothing, stored per pair: a pair's entries
        // from its first slot on (the exclusive scan of the key counts), in the row-major order of its tiles. After a
        // render that did not wait for its count there is room for every entry its lists can hold (32 MiB at most):
        // waiting for the count here would wait for all that the render's stream holds by now
        const size_t db = (size_t)w.last.n_keys * 32 * sizeof(float);
        if ((s = w.det.reserve(this, db + 16, st))) return s;
        if (db && (s = hip(hipMemsetAsync(w.det.ptr, 0, db, st), "memset entry sums"))) return s;
        det_part = (float*)w.det.ptr;
        const size_t ob = ((size_t)P * sizeof(uint32_t) + 7) / 8 * 8;
        if ((s = w.off.reserve(this, ob + 16, st))) return s;
        if ((s = w.scan.reserve(this, scan_scratch_bytes(P) + 64, st))) return s;
        launch_exclusive_scan(w.rec.count, (uint32_t*)w.off.ptr, (uint64_t*)((char*)w.off.ptr + ob), P, w.scan.ptr,
                              st);
        det_off = (const uint32_t*)w.off.ptr;
    }
    launch_blend_backward((const uint2*)w.ranges.ptr, w.last.vals, w.rec, B, w.last.grid, grad_out, auxT, auxL,
                          (float*)w.dpair.ptr, st, det_part, d.n, det_off);
    stage_end(st);
    // 3. preprocess backward -> residual-coordinate gradients
    float* dy = nullptr;
    if (want_mlp) {
        if ((s = w.dy.reserve(this, (size_t)P * kOut * sizeof(float) + 16, st))) return s;
        dy = (float*)w.dy.ptr;
        if ((s = w.groups.reserve(this, row_group_words(P) * sizeof(uint32_t), st))) return s;
    }
    stage_begin(SWF_STAGE_BWD_PREPROCESS, st);
    launch_preprocess_backward((const float*)w.dpair.ptr, w.rec, P, (flags & SWF_PAPER_DEFORM) != 0,
                               (float*)w.dbase.ptr, dy, (uint32_t*)w.groups.ptr, st);
    stage_end(st);
    // 4. MLP backward (the forward's activations; BF16 operands after a BF16 forward)
    float* dmu = nullptr;
    if (want_mlp) {
        stage_begin(SWF_STAGE_BWD_MLP, st);
        s = mlp_backward(w, d, tx, B, dy, row_groups((uint32_t*)w.groups.ptr, P), gr, bf16, st);
        last_mlp_bwd.valid = s == SWF_OK;
        last_mlp_bwd.scene = sid;
        last_mlp_bwd.B = B;
        last_mlp_bwd.n = d.n;
        last_mlp_bwd.layers = d.n_hidden;
        last_mlp_bwd.bf16 = bf16;
        stage_end(st);
        if (s) return s;
        dmu = (float*)w.dmu.ptr;
    }
    // 5. base parameters: sum over the batch, original ids
    const BaseGrads outs = {{gr->mean_x, gr->mean_y, gr->log_scale_x, gr->log_scale_y, gr->rotation,
                             gr->opacity_logit, gr->amplitude}};
    launch_base_reduce((const float*)w.dbase.ptr, dmu, d.perm, B, d.n, outs, st);
    return hip(hipGetLastError(), "backward launch");
}

}  // namespace swf

using namespace swf;

extern "C" swf_status swf_render_backward(swf_ctx* h, int32_t scene_id, const float* tx, int32_t batch, int32_t flags,
                                          const float* grad_out, const void* aux, const swf_grads* grads,
                                          void* stream) {
    Ctx* c = reinterpret_cast<Ctx*>(h);
    if (!c) return SWF_E_INVALID;
    std::lock_guard<std::recursive_mutex> lock(c->mu);
    hipSetDevice(c->device);
    return c->backward(c->ws, scene_id, tx, batch, flags, grad_out, aux, grads, (hipStream_t)stream);
}
