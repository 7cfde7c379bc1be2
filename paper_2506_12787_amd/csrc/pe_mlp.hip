// Positional encoding, FP32 deformation MLP with the fused deform + preprocess
// epilogue, and the static (no-MLP) preprocess.
//
// Deformation MLP (Sec. 4.2): residuals = F_theta(gamma(mu_hat), gamma(s_hat)).
// Layer 1 is split: its transceiver part W1s gamma(s_hat) + b1 is the same for
// every Gaussian of a query and is computed once per query (tx_features); its
// mean part W1m gamma(mu_hat) (K = 26) runs per pair. Every later layer is a
// dense 256 x 256 contraction per pair, on the FP32 matrix cores.
#include "kernels.h"
#include "swf_device.h"
#include "mlp_common.h"

namespace swf {

namespace {

// gamma(s_hat) for one query and the per-query layer-1 partial sum
// qs[b][j] = b1[j] + sum_k W1[j][26 + k] gamma_k(s_hat_b).
__global__ __launch_bounds__(256) void tx_features_kernel(const float* __restrict__ tx, const float* __restrict__ w1,
                                                          const float* __restrict__ b1, int hidden, int in_dim,
                                                          float lox, float loy, float loz, float rx, float ry,
                                                          float rz, float* __restrict__ qs,
                                                          float* __restrict__ feat_out,
                                                          uint32_t* __restrict__ status) {
    __shared__ float feat[kTxFeat];
    const int b = blockIdx.x;
    const int t = threadIdx.x;
    if (status && b == 0 && t < kStatusWords) status[t] = 0u;
    if (t < 3 * (kTxBands + 1)) {
        const int d = t % 3;
        const int k = t / 3;  // 0: identity, 1..L: band k-1
        const float v = tx[b * 3 + d];
        const float lo = d == 0 ? lox : (d == 1 ? loy : loz);
        const float rg = d == 0 ? rx : (d == 1 ? ry : rz);
        float s, e, hi, lo2;
        two_sum(v, -lo, s, e);
        div_two(s, rg, hi, lo2);
        lo2 += e / rg;
        if (k == 0) {
            feat[d] = hi + lo2;
        } else {
            float sv, cv;
            sincospi_scaled(hi, lo2, k - 1, sv, cv);
            feat[3 + 3 * (k - 1) + d] = sv;
            feat[3 + 3 * kTxBands + 3 * (k - 1) + d] = cv;
        }
    }
    __syncthreads();
    if (feat_out && t < kTxFeat) feat_out[(size_t)b * kTxFeat + t] = feat[t];
    for (int j = t; j < hidden; j += blockDim.x) {
        const float* row = w1 + (size_t)j * in_dim + kMeanFeat;
        float acc = b1[j];
        for (int k = 0; k < kTxFeat; ++k) acc = fmaf(row[k], feat[k], acc);
        qs[(size_t)b * hidden + j] = acc;
    }
}

// ---- FP32 MLP on the matrix cores ---------------------------------------------
// v_mfma_f32_16x16x4_f32 (FP32 products and sums): per layer D = W H with 16
// output units x 16 pairs per instruction and K = 4 inputs. A block of four
// waves takes kNcb column blocks of 16 pairs through the network together: wave
// w forms output tiles 4 w .. 4 w + 3 of every column block, so that a weight
// fragment (16 bytes per lane, 4 instructions per column block) is loaded once
// per block, and 4 kNcb independent sums are in flight. The hidden state lies in
// LDS as B operands: piece (cb, q), lane l = 16 g + n, holds inputs
// 16 q + 4 g + 0..3 of pair n of column block cb. The result of output tile t
// (4 registers per lane: units 16 t + 4 g + i) is, after the ReLU, exactly the
// next layer's piece t, since the fragment-major weights list their input
// columns in that order; every access is a contiguous KiB. Layer 1 takes the 26
// mean features (piece q, element j of lane group g = feature 4 (4 q + j) + g,
// zero past 26) with the per-query TX part qs[b] + b1 as its bias; the output
// layer is one tile of 16 rows, 7 used, one column block per wave. An output's
// sum runs over its inputs in the same order whatever kNcb is.
//
// Bound by the matrix cores: 3264 instructions of 32 cycles per 16 pairs. With
// whole networks per wave (weights from L2 for 16 pairs at a time, three waves
// per SIMD) the last waves of a launch ran alone on their SIMDs: 100k pairs 428
// us, now 350; 16 pairs 74 us, now 13; at full rate 81 % of the instructions' own
// time (64-pair blocks, 10 rounds).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kFWaves = 4;  // waves per block, 4 output tiles each

// Weight fragments of kAhead pieces are in flight ahead of the one in use; a layer's first ones are loaded before the
// barriers in front of it.
template <int kNcb>
constexpr int kAhead = kNcb >= 4 ? 1 : 2;

// The first fragments of the wave's tiles. wf: fragments of its first tile, kQ per tile.
template <int kNcb, int kQ>
__device__ __forceinline__ void f32_first(const float4* __restrict__ wf, int lane, float4 (&w)[kAhead<kNcb> + 1][4]) {
#pragma unroll
    for (int d = 0; d < kAhead<kNcb>; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) w[d][i] = wf[((size_t)i * kQ + d) * 64 + lane];
}

struct NoHook {
    __device__ void operator()(int) const {}
};

// acc[i][cb] += tile 4 wave + i of the layer over kQ pieces of the state; w holds the first fragments. hook(q) runs
// before piece q's instructions (the caller's own loads, in flight under them).
template <int kNcb, int kQ, typename Hook = NoHook>
__device__ __forceinline__ void f32_coop_layer(const float4* __restrict__ wf, const float4* s_h, int lane,
                                               float4 (&w)[kAhead<kNcb> + 1][4], f32x4 (&acc)[4][kNcb],
                                               Hook hook = Hook()) {
    constexpr int kA = kAhead<kNcb>;
    float4 bn[kNcb];
#pragma unroll
    for (int cb = 0; cb < kNcb; ++cb) bn[cb] = s_h[cb * 16 * 64 + lane];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        float4 b[kNcb];
#pragma unroll
        for (int cb = 0; cb < kNcb; ++cb) {
            b[cb] = bn[cb];
            if (q + 1 < kQ) bn[cb] = s_h[(cb * 16 + q + 1) * 64 + lane];
        }
        if (q + kA < kQ)
#pragma unroll
            for (int i = 0; i < 4; ++i) w[(q + kA) % (kA + 1)][i] = wf[((size_t)i * kQ + q + kA) * 64 + lane];
        hook(q);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 wi = w[q % (kA + 1)][i];
                const float wv = j == 0 ? wi.x : j == 1 ? wi.y : j == 2 ? wi.z : wi.w;
#pragma unroll
                for (int cb = 0; cb < kNcb; ++cb) {
                    const float bv = j == 0 ? b[cb].x : j == 1 ? b[cb].y : j == 2 ? b[cb].z : b[cb].w;
                    acc[i][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv, bv, acc[i][cb], 0, 0, 0);
                }
            }
        __builtin_amdgcn_sched_barrier(0);  // the loads stay where they are written
    }
}

// kMix: the queries of a mixed batch, each with its own scene (parameters, grid
// and weights). A wave's 16 pairs lie in one 384-pair MLP tile of one query
// (the tiling of the batch's tables: a query's pairs padded to whole tiles), so
// every pair of a wave takes the same weights; waves past the batch's tiles or
// past their query's pairs do nothing.
constexpr int kMixGroups = 24;  // 16-pair groups per 384-pair MLP tile of a mixed batch

// gw0: the block's first group of 16 pairs; s_h, outv, s_q (the pairs' queries): LDS for kNcb column blocks.
template <bool kMix, int kNcb>
__device__ __forceinline__ void mlp_fp32_block(const MlpArgs& a, const MixBatch& mix, int64_t gw0, float4* s_h,
                                               float (*outv)[16][8], uint32_t* s_q) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
    const int g = lane >> 4;
    // waves 0 .. kNcb - 1: the 16 pairs of column block `wave`: this lane's record row and its index p in the
    // scene; rows past the query are computed on index 0 and not written
    const MixScene* sc = nullptr;  // block-uniform: a block's pairs lie in one MLP tile of one query
    size_t row = 0;
    int p = 0;
    bool in = false;
    if constexpr (kMix) {
        static_assert(kMixGroups % kNcb == 0, "a block within one tile");
        const int gw = (int)gw0 + wave;
        const int tile = (int)gw0 / kMixGroups;
        if (tile >= mix.queries[mix.B].mlp_tile_base) return;  // block-uniform
        const int q = mix_find(mix.queries, mix.B, tile, [](const MixQuery& x) { return x.mlp_tile_base; });
        sc = &mix.scenes[mix.queries[q].scene];
        const int pb = (tile - mix.queries[q].mlp_tile_base) * (16 * kMixGroups);
        if (pb + ((int)gw0 % kMixGroups) * 16 >= sc->N) return;  // block-uniform: no pair in the block
        p = pb + (gw % kMixGroups) * 16 + (lane & 15);
        in = wave < kNcb && p < sc->N;
        row = (size_t)mix.queries[q].pair_base + p;
        if ((int)threadIdx.x < kNcb * 16) s_q[threadIdx.x] = (uint32_t)q;
    } else {
        const size_t total = (size_t)a.N * a.B;
        row = ((size_t)gw0 + wave) * 16 + (lane & 15);
        in = wave < kNcb && row < total;
        p = in ? (int)(row % a.N) : 0;
        if (wave < kNcb && lane < 16) s_q[wave * 16 + lane] = in ? (uint32_t)(row / a.N) : 0u;
    }
    if (!in) p = 0;
    if (wave < kNcb) {
        float f[kMeanFeat];
        if constexpr (kMix)
            mean_features(sc->mx[p], sc->my[p], sc->W, sc->H, f);
        else
            mean_features(a.mx[p], a.my[p], a.sW, a.sH, f);
        float x[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float v0 = 4 * c < kMeanFeat ? f[4 * c] : 0.0f;
            const float v1 = 4 * c + 1 < kMeanFeat ? f[4 * c + 1] : 0.0f;
            const float v2 = 4 * c + 2 < kMeanFeat ? f[4 * c + 2] : 0.0f;
            const float v3 = 4 * c + 3 < kMeanFeat ? f[4 * c + 3] : 0.0f;
            x[c] = g == 0 ? v0 : (g == 1 ? v1 : (g == 2 ? v2 : v3));
        }
        s_h[(wave * 16) * 64 + lane] = make_float4(x[0], x[1], x[2], x[3]);
        s_h[(wave * 16 + 1) * 64 + lane] = make_float4(x[4], x[5], x[6], x[7]);
    }
    // the network's weights: the batch's scene (kMix, four hidden layers) or the launch's
    const float* frag = kMix ? sc->f32_frag : nullptr;
    const int n_mid = kMix ? 3 : a.n_mid;
    const float4* wf1 = kMix ? reinterpret_cast<const float4*>(frag) : a.wf1;
    const float4* wfo = kMix ? reinterpret_cast<const float4*>(frag + frag_out_at(4)) : a.wfo;
    const float* bo16 = kMix ? frag + frag_out_at(4) + kFragOut : a.bo16;
    float4 w[kAhead<kNcb> + 1][4];
    wf1 += (size_t)4 * wave * 2 * 64;
    f32_first<kNcb, 2>(wf1, lane, w);
    __syncthreads();
    f32x4 acc[4][kNcb];
    // the sums through the ReLU into the state (and, kept for the backward, to activation `lay`)
    const auto leave = [&](int lay) {
        float* st = kMix ? nullptr : a.act_out[lay];
        const size_t row0 = (size_t)gw0 * 16, total = kMix ? 0 : (size_t)a.N * a.B;
        __syncthreads();  // every wave has read the layer's input
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int cb = 0; cb < kNcb; ++cb) {
                const int t = 4 * wave + i;
                const float4 h = make_float4(fmaxf(acc[i][cb][0], 0.0f), fmaxf(acc[i][cb][1], 0.0f),
                                             fmaxf(acc[i][cb][2], 0.0f), fmaxf(acc[i][cb][3], 0.0f));
                s_h[(cb * 16 + t) * 64 + lane] = h;
                const size_t r = row0 + cb * 16 + (lane & 15);
                if (st && r < total)  // one contiguous KiB per column block
                    __builtin_nontemporal_store(f32x4{h.x, h.y, h.z, h.w},
                                                reinterpret_cast<f32x4*>(st + piece_at((int64_t)r, t, g)));
            }
        __syncthreads();
    };
#pragma unroll
    for (int cb = 0; cb < kNcb; ++cb) {
        const float* qrow = a.qs + (size_t)s_q[cb * 16 + (lane & 15)] * 256;  // the layer's bias (the TX term)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 b4 = *reinterpret_cast<const float4*>(qrow + 16 * (4 * wave + i) + 4 * g);
            acc[i][cb] = f32x4{b4.x, b4.y, b4.z, b4.w};
        }
    }
    f32_coop_layer<kNcb, 2>(wf1, s_h, lane, w, acc);
#pragma unroll 1
    for (int l = 0; l < n_mid; ++l) {
        const float4* wh = (kMix ? reinterpret_cast<const float4*>(frag + frag_hidden_at(l + 1)) : a.wfh[l]) +
                           (size_t)4 * wave * 16 * 64;
        const float* bh = kMix ? sc->bias_h[l] : a.bh[l];
        f32_first<kNcb, 16>(wh, lane, w);
        float4 b4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b4[i] = *reinterpret_cast<const float4*>(bh + 16 * (4 * wave + i) + 4 * g);
        __builtin_amdgcn_sched_barrier(0);
        leave(l);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int cb = 0; cb < kNcb; ++cb) acc[i][cb] = f32x4{b4[i].x, b4[i].y, b4[i].z, b4[i].w};
        f32_coop_layer<kNcb, 16>(wh, s_h, lane, w, acc);
    }
    leave(n_mid);
    if (wave >= kNcb) return;  // no barrier follows for these waves' outputs
    // output layer: lane l holds outputs 4 (l / 16) + i of pair l % 16
    f32x4 o = f32x4{bo16[4 * g], bo16[4 * g + 1], bo16[4 * g + 2], bo16[4 * g + 3]};
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const float4 w = wfo[q * 64 + lane], b = s_h[(wave * 16 + q) * 64 + lane];
        o = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, b.x, o, 0, 0, 0);
        o = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, b.y, o, 0, 0, 0);
        o = __builtin_amdgcn_mfma_f32_16x16x4f32(w.z, b.z, o, 0, 0, 0);
        o = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w, b.w, o, 0, 0, 0);
    }
    if (g < 2) {
#pragma unroll
        for (int i = 0; i < 4; ++i) outv[wave][lane & 15][4 * g + i] = o[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < 16 && in) {  // lanes 0..15 hold the wave's 16 pairs (lane l: pair l)
        if constexpr (kMix)
            mix_epilogue(*sc, a, row, p, outv[wave][lane]);
        else
            deform_epilogue(a, row, p, outv[wave][lane]);
    }
}

// Blocks [0, n4) take 64 pairs each, the others 16 (launch_mlp_fp32's split).
template <bool kMix>
__global__ __launch_bounds__(64 * kFWaves, 2) void mlp_fp32_kernel(MlpArgs a, MixBatch mix, int n4) {
    __shared__ __attribute__((aligned(16))) float4 s_h[kFWaves * 16 * 64];
    __shared__ float outv[kFWaves][16][8];
    __shared__ uint32_t s_q[kFWaves * 16];
    const int64_t b = blockIdx.x;
    if (kMix || b < n4)  // block-uniform
        mlp_fp32_block<kMix, kFWaves>(a, mix, b * kFWaves, s_h, outv, s_q);
    else if constexpr (!kMix)
        mlp_fp32_block<false, 1>(a, mix, (int64_t)n4 * kFWaves + (b - n4), s_h, outv, s_q);
}

// Input gradient of a 256 x 256 layer of the FP32 backward on the same matrix
// cores: out[p][i] = [act[p][i] > 0] sum_o W[o][i] dz[p][o], the layer function
// above with W^T as its weights (fragment-major, packed by pack_wt_kernel) and
// no bias, over the listed groups, two to a block. A wave brings 16 rows into the
// state: lane l = 16 g + r loads piece q (inputs 16 q + 4 g + 0..3) of row r as
// 16 bytes; masked output tile t (units 16 t + 4 g + i) goes out as 16 bytes.
// A block's 16 loads per lane go out together and the ReLU masks are loaded under
// the matrix instructions, so that little but those is waited for: 160k pairs 202
// us (230 with each load in a branch of its own, 247 with a layer per wave; the
// instructions' own time is 146, the bytes' 103).
__global__ __launch_bounds__(64 * kFWaves, 2) void dz_f32_kernel(const float* __restrict__ dz,
                                                                 const float4* __restrict__ wt,
                                                                 const float* __restrict__ act, int64_t P,
                                                                 RowGroups rg, float* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) float4 s_h[kFWaves * 16 * 64];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
    const int g = lane >> 4;
    // the block's listed groups of 32 rows: two waves each
    static_assert(kRowGroup == 32 && kFWaves == 4, "two groups per block");
    const uint32_t ng = *rg.count, gi = 2 * blockIdx.x + (wave >> 1);
    if (2 * blockIdx.x >= ng) return;  // block-uniform: no rows
    const int64_t p0 = gi < ng ? (int64_t)rg.list[gi] * kRowGroup + 16 * (wave & 1) : P;
    const int64_t row = p0 + (lane & 15);
    {
        const bool in = row < P;
        const float* px = dz + piece_at(in ? row : 0, 0, g);  // a row that is none reads row 0 and counts zero
        float4 x[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) x[q] = *reinterpret_cast<const float4*>(px + 256 * q);
#pragma unroll
        for (int q = 0; q < 16; ++q)
            s_h[(wave * 16 + q) * 64 + lane] = in ? x[q] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    __syncthreads();
    // rows of the column blocks: two per listed group
    wt += (size_t)4 * wave * 16 * 64;
    float4 w[kAhead<kFWaves> + 1][4];
    f32_first<kFWaves, 16>(wt, lane, w);
    int64_t rows[kFWaves];
#pragma unroll
    for (int cb = 0; cb < kFWaves; ++cb) {
        const uint32_t k = 2 * blockIdx.x + (cb >> 1);
        const int64_t r = k < ng ? (int64_t)rg.list[k] * kRowGroup + 16 * (cb & 1) + (lane & 15) : P;
        rows[cb] = r < P ? r : -1;
    }
    f32x4 acc[4][kFWaves];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int cb = 0; cb < kFWaves; ++cb) acc[i][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // under the instructions of piece q: the activations of output tile q / 4, column block q % 4, kept as 4 bits
    // (a row that is none reads row 0 and is not stored)
    const float* pm[kFWaves];
#pragma unroll
    for (int cb = 0; cb < kFWaves; ++cb) pm[cb] = act + piece_at(max(rows[cb], (int64_t)0), 4 * wave, g);
    float4 mk = make_float4(0.f, 0.f, 0.f, 0.f);
    uint64_t bits = 0;
    const auto keep = [&](int q) {
        const uint32_t b = (mk.x > 0.f ? 1u : 0u) | (mk.y > 0.f ? 2u : 0u) | (mk.z > 0.f ? 4u : 0u) |
                           (mk.w > 0.f ? 8u : 0u);
        bits |= (uint64_t)b << (4 * q);
    };
    f32_coop_layer<kFWaves, 16>(wt, s_h, lane, w, acc, [&](int q) {
        if (q) keep(q - 1);
        mk = *reinterpret_cast<const float4*>(pm[q & 3] + 256 * (q >> 2));
    });
    keep(15);
#pragma unroll
    for (int cb = 0; cb < kFWaves; ++cb) {
        if (rows[cb] < 0) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t m = (uint32_t)(bits >> (4 * (4 * i + cb)));
            *reinterpret_cast<float4*>(out + piece_at(rows[cb], 4 * wave + i, g)) =
                make_float4(m & 1u ? acc[i][cb][0] : 0.0f, m & 2u ? acc[i][cb][1] : 0.0f,
                            m & 4u ? acc[i][cb][2] : 0.0f, m & 8u ? acc[i][cb][3] : 0.0f);
        }
    }
}

// W^T of a 256 x 256 layer (W row-major [out][in]) in the fragment order of
// f32_coop_layer: fragment q of output tile t, lane l = 16 g + r, element j
// holds W^T[16 t + r][16 q + 4 g + j] = W[16 q + 4 g + j][16 t + r].
__global__ void pack_wt_kernel(const float* __restrict__ w, float* __restrict__ wt) {
    const int e = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (e >= 65536) return;
    const int t = e / 4096, q = (e / 256) % 16, l = (e / 4) % 64, j = e % 4;
    wt[e] = w[(size_t)(16 * q + 4 * (l >> 4) + j) * 256 + 16 * t + (l & 15)];
}

__global__ void preprocess_static_kernel(MlpArgs a) {
    const size_t row = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)a.N * a.B;
    if (row >= total) return;
    const int p = (int)(row % a.N);
    PairOut o;
    if (p < a.n_live) {
        o = preprocess_pair(a.mx[p], a.my[p], 0.f, 0.f, a.lsx[p], a.lsy[p], a.rot[p], a.logit[p], a.amp[p], a.W, a.H,
                            a.TW, a.TH, a.inv_tile, a.wrap, a.sx, a.sy);
    } else {
        o.geo = make_float4(0, 0, 0, 0);
        o.wm = make_float4(0, 0, 0, 0);
        o.oa = make_float2(0, 0);
        o.rect_x = o.rect_y = 0;
        o.count = 0;
    }
    write_record(a.rec, row, o);
}

__global__ void permute_delta_kernel(const float* __restrict__ src, const uint32_t* __restrict__ perm, int B, int n,
                                     float* __restrict__ dst) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)B * n) return;
    const size_t b = i / n, p = i % n;
    const size_t o = b * n + perm[p];
#pragma unroll
    for (int k = 0; k < kOut; ++k) dst[o * kOut + k] = src[i * kOut + k];
}

struct Ptr7 {
    const float* s[7];
    float* d[7];
};

__global__ void gather_params_kernel(Ptr7 p, const uint32_t* __restrict__ perm, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t src = perm[i];
#pragma unroll
    for (int k = 0; k < 7; ++k) p.d[k][i] = p.s[k][src];
}

}  // namespace

void launch_gather_params(const float* const* src, const uint32_t* perm, int n, float* const* dst, hipStream_t st) {
    Ptr7 p;
    for (int k = 0; k < 7; ++k) {
        p.s[k] = src[k];
        p.d[k] = dst[k];
    }
    if (n > 0) gather_params_kernel<<<(n + 255) / 256, 256, 0, st>>>(p, perm, n);
}

void launch_tx_features(const DevScene& s, const float* tx, int B, float* qs, uint32_t* status, hipStream_t st,
                        float* feat_out) {
    const float rx = s.room_hi[0] - s.room_lo[0], ry = s.room_hi[1] - s.room_lo[1], rz = s.room_hi[2] - s.room_lo[2];
    tx_features_kernel<<<B, 256, 0, st>>>(tx, s.w[0], s.b[0], s.hidden, s.in_dim, s.room_lo[0], s.room_lo[1],
                                          s.room_lo[2], rx, ry, rz, qs, feat_out, status);
}

void launch_mlp_fp32(const DevScene& s, const float* qs, int B, const Grid& g, bool paper_mask, const Records& r,
                     float* delta_out, hipStream_t st, float* const* act_out) {
    MlpArgs a = make_args(s, qs, B, g, paper_mask, r, delta_out);
    if (act_out)
        for (int l = 0; l < s.n_hidden && l < 8; ++l) a.act_out[l] = act_out[l];
    const size_t groups = ((size_t)s.n * B + 15) / 16;
    if (!groups) return;
    // Whole rounds of 64-pair blocks over the compute units (57 us each), then the rest: 64-pair blocks take one round
    // more however few they are, 16-pair blocks one shorter round (24 us) for as many groups as there are compute
    // units, with four times the weight loads. One render of n Gaussians, us (16-pair / 64-pair blocks for the rest):
    // n = 16: 48 / 83; 4,000: 69 / 103; 8,000: 94 / 112; 12,000: 117 / 117; 20,000: 142 / 174; 100,000: 414 / 446.
    const int64_t cus = n_compute_units();
    int64_t n4 = (int64_t)groups / (4 * cus) * cus, rest = (int64_t)groups - 4 * n4;
    if (rest > 2 * cus) {
        n4 += (rest + 3) / 4;
        rest = 0;
    }
    mlp_fp32_kernel<false><<<(unsigned)(n4 + rest), 64 * kFWaves, 0, st>>>(a, MixBatch{}, (int)n4);
}

void launch_mix_mlp_fp32(const MixBatch& m, const float* qs, const Records& r, int64_t pair_cap, int B_cap,
                         hipStream_t st, bool paper_mask, bool wrap) {
    // every 384-pair tile the batch can hold (its pairs, each query padded to whole tiles)
    const int64_t tiles = (pair_cap + 383) / 384 + B_cap;
    const int64_t blocks = (tiles * kMixGroups + kFWaves - 1) / kFWaves;
    MlpArgs a{};
    a.qs = qs;
    a.rec = r;
    a.inv_tile = 1.0f / 16.0f;
    a.paper_mask = paper_mask ? 1 : 0;
    a.wrap = wrap ? 1 : 0;
    if (blocks > 0) mlp_fp32_kernel<true><<<(unsigned)blocks, 64 * kFWaves, 0, st>>>(a, m, 0);
}

void launch_preprocess_static(const DevScene& s, int B, const Grid& g, const Records& r, hipStream_t st) {
    const MlpArgs a = make_args(s, nullptr, B, g, false, r, nullptr);
    const size_t total = (size_t)s.n * B;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (blocks) preprocess_static_kernel<<<blocks, 256, 0, st>>>(a);
}

void launch_permute_delta(const float* delta_sorted, const uint32_t* perm, int B, int n, float* delta_out,
                          hipStream_t st) {
    const size_t total = (size_t)B * n;
    if (total) permute_delta_kernel<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(delta_sorted, perm, B, n, delta_out);
}

void launch_pack_wt(const float* w, float* wt, hipStream_t st) { pack_wt_kernel<<<256, 256, 0, st>>>(w, wt); }

void launch_dz_f32(const float* dz, const float* wt, const float* act, int64_t P, const RowGroups& rg, float* out,
                   hipStream_t st) {
    if (P > 0)
        dz_f32_kernel<<<(unsigned)((P + 63) / 64), 64 * kFWaves, 0, st>>>(dz, reinterpret_cast<const float4*>(wt), act,
                                                                          P, rg, out);
}

}  // namespace swf
