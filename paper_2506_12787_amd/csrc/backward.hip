// Backward pass of the render path: blend -> preprocess -> deformation MLP.
//
// Blend backward (Sec. 3.2 blending rule, differentiated): per (query, tile)
// workgroup, each pixel replays its transmittance back to front from the
// stored final T and last-contributor index, T_before = T_after / (1 - alpha)
// (alpha <= 0.99 so the divisor is >= 0.01), and accumulates
//   dC/damp_i   = alpha_i T_i
//   dC/dalpha_i = amp_i T_i - S_i / (1 - alpha_i),  S_i = sum_{j>i} amp_j alpha_j T_j
// through alpha = min(0.99, o exp(-q/2)) (zero derivative when clamped),
// q = |M d|^2, into per-pair gradients of (mean, M, opacity, amplitude).
// Per entry the 64 lanes of a wave are reduced before one atomic per value.
// With 16x16 tiles a wave skips the entries that miss the cutoff on all of its
// pixels.
//
// Preprocess backward maps d(M, opacity) to the 7 residual coordinates
// (d_mean, d_log_scale, d_rotation, d_logit, d_amp); the MLP backward is a
// chain of row-parallel products (dZ_{l-1} = (dZ_l W_l) . [H_{l-1} > 0]) and
// split-K weight-gradient reductions (dW_l = dZ_l^T H_{l-1}) in FP32.
#include <cmath>

#include "cull.h"
#include "kernels.h"
#include "swf_device.h"

namespace swf {

namespace {

__device__ __forceinline__ unsigned lane_id() { return threadIdx.x & 63u; }

// v of the lane that the DPP control names, in the rows and banks of the masks
// (elsewhere old).
template <int kCtrl, int kBank>
__device__ __forceinline__ float dpp(float old, float v) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), kCtrl, 0xf, kBank, kBank == 0xf));
}

// Wave sums of 8 values at once: halving exchanges with lanes l ^ 1, l ^ 2 and
// l ^ 4 leave each lane one value summed over 8 lanes, sums with l ^ 8, l ^ 16 and
// l ^ 32 finish it. All in registers (DPP and lane swaps; every lane of the wave is
// active): as shuffles through LDS, ten in a row, they were a quarter of the blend
// backward's time. (Halving with l ^ 32, 16 and 8 first takes a third fewer
// instructions, but adds in another order: a gradient that is rounded to BF16
// further on then falls the other way here and there.) Lane l < 8 returns the total
// of value index 4 (l & 1) + 2 ((l >> 1) & 1) + ((l >> 2) & 1).
__device__ __forceinline__ float wave_sum8(float (&a)[8]) {
    const unsigned l = lane_id();
    {
        const bool hi = l & 1u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float send = hi ? a[k] : a[k + 4], keep = hi ? a[k + 4] : a[k];
            a[k] = keep + dpp<0xb1, 0xf>(0.f, send);  // quad_perm 1,0,3,2
        }
    }
    {
        const bool hi = l & 2u;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float send = hi ? a[k] : a[k + 2], keep = hi ? a[k + 2] : a[k];
            a[k] = keep + dpp<0x4e, 0xf>(0.f, send);  // quad_perm 2,3,0,1
        }
    }
    float v;
    {
        const bool hi = l & 4u;
        const float send = hi ? a[0] : a[1], keep = hi ? a[1] : a[0];
        // row_shl:4 into banks 0 and 2, row_shr:4 into 1 and 3
        v = keep + dpp<0x114, 0xa>(dpp<0x104, 0x5>(send, send), send);
    }
    v += dpp<0x128, 0xf>(0.f, v);  // row_ror:8
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

// With 16x16 tiles each wave (an 8x8 quadrant) walks only the entries that can
// reach the cutoff on its rectangle (the forward kernel's culling): the others
// leave every one of its pixels unchanged.
// Bound by vector issue (80 % of the time): per entry and wave about 22
// instructions to find that no pixel takes it, 80 more if one does. Hence one
// reciprocal for a pixel's two quotients, the opacity's taken when the entry is
// staged, and indices broadcast from a register. 50k Gaussians, 16 positions of
// 90 x 360, 1.5M entries evaluated: 233 us (346 with LDS shuffles, three
// divisions and nested branches; every wave's sums are the same bit for bit).
// kWrap: periodic azimuth, as in the forward kernel (same staged image, same
// displacement, same culling exemption), so that every decision replays exactly.
// kDet: instead of adding into dpair, each wave writes its 8 sums of an entry
// to part[slot * 32 + wave * 8 + k] (zeroed beforehand), slot = the pair's
// first slot (det_off: the exclusive scan of the key counts) + the tile's
// row-major index in the pair's rectangle; det_reduce_kernel then sums each
// pair's slots in that order.
template <int TILE, bool kWrap = false, bool kDet = false>
__global__ __launch_bounds__(TILE* TILE) void blend_backward_kernel(
    const uint2* __restrict__ ranges, const uint32_t* __restrict__ vals, const float4* __restrict__ geo,
    const float4* __restrict__ wm, const float2* __restrict__ oa, int H, int W, int TW, int tiles,
    const float* __restrict__ grad_out, const float* __restrict__ aux_T, const uint32_t* __restrict__ aux_last,
    float* __restrict__ dpair, float* __restrict__ part = nullptr, const uint2* __restrict__ rect = nullptr,
    const uint32_t* __restrict__ det_off = nullptr) {
    constexpr int kN = TILE * TILE;
    constexpr bool kCull = TILE == 16;
    constexpr int kWaves = kN / 64;
    __shared__ float2 s_pos[kN];
    __shared__ float4 s_wm[kN];
    __shared__ float4 s_oa[kN];  // opacity, amplitude, 1 / opacity
    __shared__ uint32_t s_v[kN];
    __shared__ uint32_t s_slot[kDet ? kN : 1];
    __shared__ uint8_t s_strip[kCull ? kN : 1];
    __shared__ uint16_t s_idx[kCull ? kWaves : 1][kN];
    __shared__ uint32_t s_max;

    const int gtile = blockIdx.x;
    const int b = gtile / tiles;
    const int t = gtile - b * tiles;
    const int tx = t % TW, ty = t / TW;
    // culled 16x16 tiles: wave w covers the 8x8 quadrant (w & 1, w >> 1)
    const int wq = (int)(threadIdx.x >> 6), lq = (int)(threadIdx.x & 63);
    const int lx = kCull ? (wq & 1) * 8 + (lq & 7) : (int)threadIdx.x % TILE;
    const int ly = kCull ? (wq >> 1) * 8 + (lq >> 3) : (int)threadIdx.x / TILE;
    const int px = tx * TILE + lx, py = ty * TILE + ly;
    const bool inside = px < W && py < H;
    const int bx0 = (tx * TILE) & ~63, by0 = (ty * TILE) & ~63;
    const float x0 = (float)bx0, y0 = (float)by0;
    const float fx = (float)(px - bx0), fy = (float)(py - by0);
    const float Wf = kWrap ? (float)W : 0.0f, rw = kWrap ? 1.0f / (float)W : 0.0f;
    const float cx = (float)(tx * TILE - bx0) + 0.5f * (float)(TILE - 1);
    const uint2 rg = ranges[gtile];

    float T = 1.0f, G = 0.0f;
    uint32_t last = 0;
    if (inside) {
        const size_t pix = (size_t)b * H * W + (size_t)py * W + px;
        G = grad_out[pix];
        if (G != 0.0f) {
            T = aux_T[pix];
            last = aux_last[pix];
        }
    }
    if (threadIdx.x == 0) s_max = 0;
    __syncthreads();
    if (last) atomicMax(&s_max, last);
    __syncthreads();
    // never past the tile's list, even for an aux that does not belong to these lists
    const int lmax = (int)min(s_max, rg.y - rg.x);
    float S = 0.0f;

    // Straight-line, one pixel per lane: a pixel that the entry leaves unchanged selects zeros (of the displacement's
    // image too, so that an overflow there stays its own).
    auto entry = [&](int beg, int jj) {
        const float4 m = s_wm[jj], o = s_oa[jj];  // o: opacity, amplitude, 1 / opacity
        float dx, dy, u, w;
        const float q = kWrap ? blend_q_wrap(fx, fy, s_pos[jj], m, Wf, rw, dx, dy, u, w)
                              : blend_q(fx, fy, s_pos[jj], m, dx, dy, u, w);
        const float e = blend_raw_alpha(q, 1.0f), raw = o.x * e;  // as blend_raw_alpha(q, o.x)
        const float a = fminf(kAlphaMax, raw);
        const bool contrib = beg + jj < (int)last && q <= kQMax && a >= kAlphaMin;
        if (__ballot(contrib) == 0ull) return;
        float gv[8];
        {
            // Quotients by om (in [0.01, 1] where it counts) and the opacity: a product with the refined reciprocal and
            // one correction, which rounds as the division does
            const float om = 1.0f - a, r0 = __builtin_amdgcn_rcpf(om), r = fmaf(fmaf(-om, r0, 1.0f), r0, r0);
            const float Tq = T * r, Tb = fmaf(fmaf(-om, Tq, T), r, Tq);  // T / om
            const float Sq = S * r, So = __builtin_amdgcn_div_fixupf(fmaf(fmaf(-om, Sq, S), r, Sq), om, S);  // S / om
            const float dC_da = o.y * Tb - So;
            gv[7] = contrib ? G * a * Tb : 0.f;
            const bool moves = contrib && !(raw > kAlphaMax);
            const float ga = G * dC_da;
            const float eq = raw * o.z, ro = fmaf(fmaf(-o.x, eq, raw), o.z, eq);  // raw / opacity = exp(-q/2)
            gv[6] = moves ? ga * ro : 0.f;           // d alpha / d opacity
            const float dq = moves ? -ga * a : 0.f;  // twice d alpha / d q = -alpha / 2
            const float du = dq * (moves ? u : 0.f), dw = dq * (moves ? w : 0.f);
            gv[0] = -(du * m.x + dw * m.z);
            gv[1] = -(du * m.y + dw * m.w);
            gv[2] = du * dx;
            gv[3] = du * dy;
            gv[4] = dw * dx;
            gv[5] = dw * dy;
            S = contrib ? fmaf(o.y * a, Tb, S) : S;
            T = contrib ? Tb : T;
        }
        const float v = wave_sum8(gv);
        const unsigned l = lane_id();
        if (l < 8u && v != 0.0f) {
            const int k = 4 * (int)(l & 1u) + 2 * (int)((l >> 1) & 1u) + (int)((l >> 2) & 1u);
            if constexpr (kDet)
                part[(size_t)s_slot[jj] * 32 + (size_t)wq * 8 + k] = v;
            else
                atomicAdd(dpair + (size_t)s_v[jj] * 8 + k, v);
        }
    };

    for (int end = lmax; end > 0; end -= kN) {
        const int beg = end > kN ? end - kN : 0;
        __syncthreads();
        {
            const int j = beg + (int)threadIdx.x;
            if (j < end) {
                const uint32_t v = vals[rg.x + j];
                const float4 g = geo[v];
                const float2 pos =
                    kWrap ? staged_mean(g, x0, y0, Wf, cx) : make_float2((g.x - x0) + g.z, (g.y - y0) + g.w);
                const float4 m = wm[v];
                s_pos[threadIdx.x] = pos;
                s_wm[threadIdx.x] = m;
                const float2 o = oa[v];
                s_oa[threadIdx.x] = make_float4(o.x, o.y, 1.0f / o.x, 0.0f);
                s_v[threadIdx.x] = v;
                if constexpr (kDet) {  // this tile's slot of the pair: row-major in its (possibly wrapped) rectangle
                    const uint2 rr = rect[v];
                    const int rx0 = (int)(rr.x & 0xffff), rx1 = (int)(rr.x >> 16), ry0 = (int)(rr.y & 0xffff);
                    const int rw = rx1 >= rx0 ? rx1 - rx0 + 1 : TW - rx0 + rx1 + 1;
                    const int cx = tx >= rx0 ? tx - rx0 : tx - rx0 + TW;
                    s_slot[threadIdx.x] = det_off[v] + (uint32_t)((ty - ry0) * rw + cx);
                }
                if (kCull)
                    s_strip[threadIdx.x] =
                        (kWrap && fabsf(pos.x - cx) > 0.5f * Wf - (float)TILE)
                            ? (uint8_t)0xf
                            : (uint8_t)wave_quads_mask(m, pos, (float)(tx * TILE - bx0), (float)(ty * TILE - by0),
                                                       kQMax);
            }
        }
        __syncthreads();
        const int cnt = end - beg;
        if (kCull) {
            const int wv = threadIdx.x >> 6;
            uint16_t* idx = s_idx[wv];
            int nlist = 0;
#pragma unroll
            for (int c = 0; c < kWaves; ++c) {
                const int jl = c * 64 + (int)lane_id();
                const bool f = jl < cnt && ((s_strip[jl] >> wv) & 1u);
                const uint64_t bal = __ballot(f);
                if (f) idx[nlist + __popcll(bal & ((1ull << lane_id()) - 1ull))] = (uint16_t)jl;
                nlist += __popcll(bal);
            }
            __builtin_amdgcn_wave_barrier();
            for (int n0 = nlist - 1; n0 >= 0; n0 -= 64) {  // 64 indices in a register at a time, back to front
                const int mine = (int)idx[max(n0 - (int)lane_id(), 0)], cnt64 = min(n0 + 1, 64);
                for (int n = 0; n < cnt64; ++n) entry(beg, __builtin_amdgcn_readlane(mine, n));
            }
        } else {
            for (int jj = cnt - 1; jj >= 0; --jj) entry(beg, jj);
        }
    }
}

// Deterministic gradient sums: pair i adds, for every tile of its rectangle in
// row-major order (a wrapped rectangle's columns from tx0 on), the four waves'
// sums of its entry there, which lie together from the pair's first slot on.
__global__ void det_reduce_kernel(const uint32_t* __restrict__ count, const uint32_t* __restrict__ det_off,
                                  const float* __restrict__ part, int64_t P, float* __restrict__ dpair) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P) return;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const uint32_t c = count[i];
    const float4* e = reinterpret_cast<const float4*>(part + (size_t)(c ? det_off[i] : 0u) * 32);
    for (uint32_t k = 0; k < c; ++k)  // the pair's tiles in row-major order, then the 4 waves of each
#pragma unroll
        for (int wv = 0; wv < 4; ++wv) {
            const float4 a = e[(size_t)k * 8 + 2 * wv], b = e[(size_t)k * 8 + 2 * wv + 1];
            acc[0] += a.x;
            acc[1] += a.y;
            acc[2] += a.z;
            acc[3] += a.w;
            acc[4] += b.x;
            acc[5] += b.y;
            acc[6] += b.z;
            acc[7] += b.w;
        }
#pragma unroll
    for (int k = 0; k < 8; ++k) dpair[i * 8 + k] = acc[k];
}

// d(mean, M, opacity, amp) -> d(residual coordinates); the unmasked result
// feeds the base parameters, the masked one (paper mode zeroes 2..4) the MLP.
//
// With dy also which rows (pairs) have a gradient at all: bits[w] bit k is set
// if row 32 w + k has a non-zero dy, or a non-finite residual (whose hidden
// activations may not be finite: a zero gradient times those is no zero), and
// groups[block] counts the block's groups of 32 rows with a set bit. Rows
// behind the pixels' termination depth or outside every pixel's cutoff have
// none: at N = 50k, 90 x 360, five of six.
__global__ __launch_bounds__(256) void preprocess_backward_kernel(
    const float* __restrict__ dpair, const float4* __restrict__ wm, const float2* __restrict__ oa,
    const uint32_t* __restrict__ count, const uint2* __restrict__ rect, int64_t P, int paper_mask,
    float* __restrict__ dbase, float* __restrict__ dy, uint32_t* __restrict__ bits, uint32_t* __restrict__ groups) {
    __shared__ uint32_t s_n;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = i < P;
    float r[kOut] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    bool live = false;
    if (in && count[i] == 0) live = rect[i].y == kCullNonFinite;
    if (in && count[i]) {
        const float* g = dpair + i * 8;
        const float4 m = wm[i];
        const float op = oa[i].x;
        r[0] = g[0];
        r[1] = g[1];
        r[2] = -(g[2] * m.x + g[3] * m.y);
        r[3] = -(g[4] * m.z + g[5] * m.w);
        r[4] = -g[2] * m.y + g[3] * m.x - g[4] * m.w + g[5] * m.z;
        r[5] = g[6] * op * (1.0f - op);
        r[6] = g[7];
    }
    if (in) {
#pragma unroll
        for (int k = 0; k < kOut; ++k) dbase[i * kOut + k] = r[k];
    }
    if (!dy) return;  // kernel-uniform
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    if (in) {
#pragma unroll
        for (int k = 0; k < kOut; ++k) {
            const float v = (paper_mask && k >= 2 && k <= 4) ? 0.f : r[k];
            dy[i * kOut + k] = v;
            live = live || !(v == 0.f);
        }
    }
    const uint64_t m = __ballot(live);
    if ((lane_id() & 31u) == 0 && in) {
        const uint32_t w = lane_id() ? (uint32_t)(m >> 32) : (uint32_t)m;
        bits[i >> 5] = w;
        if (w) atomicAdd(&s_n, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) groups[blockIdx.x] = s_n;
}

// The groups of 32 rows with a gradient, in row order: list[0 .. count). Block
// k takes 1024 groups (128 blocks of the pass above, whose counts give its
// first position).
__global__ __launch_bounds__(1024) void row_groups_kernel(const uint32_t* __restrict__ bits,
                                                          const uint32_t* __restrict__ groups, int64_t n_groups,
                                                          uint32_t* __restrict__ list, uint32_t* __restrict__ count) {
    __shared__ uint32_t s_sum[16];
    const int w = (int)threadIdx.x >> 6;
    uint32_t before = 0;
    for (int64_t j = threadIdx.x; j < (int64_t)blockIdx.x * 128; j += 1024) before += groups[j];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
    if (lane_id() == 0) s_sum[w] = before;
    __syncthreads();
    uint32_t base = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) base += s_sum[k];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    const bool f = i < n_groups && bits[i] != 0u;
    const uint64_t m = __ballot(f);
    if (lane_id() == 0) s_sum[w] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t all = base;
    for (int k = 0; k < 16; ++k) {
        if (k < w) base += s_sum[k];
        all += s_sum[k];
    }
    if (f) list[base + (uint32_t)__popcll(m & ((1ull << lane_id()) - 1ull))] = (uint32_t)i;
    if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) *count = all;
}

// Base-parameter gradients: sum over the batch, scatter to original ids.
__global__ void base_reduce_kernel(const float* __restrict__ dbase, const float* __restrict__ dmu_pe,
                                   const uint32_t* __restrict__ perm, int B, int N, BaseGrads out) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    float s[kOut] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int b = 0; b < B; ++b) {
        const float* r = dbase + ((size_t)b * N + p) * kOut;
#pragma unroll
        for (int k = 0; k < kOut; ++k) s[k] += r[k];
    }
    if (dmu_pe) {
        s[0] += dmu_pe[(size_t)p * 2];
        s[1] += dmu_pe[(size_t)p * 2 + 1];
    }
    const uint32_t id = perm[p];
#pragma unroll
    for (int k = 0; k < kOut; ++k)
        if (out.p[k]) out.p[k][id] = s[k];
}

__device__ __forceinline__ float4 load4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 load4(const __bf16* p) {
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xffff0000u));
}

// Column sums of a row-major [rows x cols] matrix of many rows (cols % 4 == 0),
// in two stages: part[y][c] over row block y (4 consecutive columns per thread,
// 64 threads over 256 columns, 4 row groups per block summed through LDS in a
// fixed order), then out[c].
__global__ __launch_bounds__(256) void colsum4_stage1_kernel(const float* __restrict__ A, int64_t rows, int64_t cols,
                                                             int64_t rpb, float* __restrict__ part) {
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * 256 + tx * 4;
    const int64_t r0 = (int64_t)blockIdx.y * rpb, r1 = min(rows, r0 + rpb);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < cols) {
#pragma unroll 4
        for (int64_t r = r0 + ty; r < r1; r += 4) {
            const float4 v = load4(A + r * cols + c);
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
    }
    __shared__ float4 red[4][64];
    red[ty][tx] = s;
    __syncthreads();
    if (ty != 0 || c >= cols) return;
    float4 t = red[0][tx];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        const float4 u = red[k][tx];
        t.x += u.x;
        t.y += u.y;
        t.z += u.z;
        t.w += u.w;
    }
    *reinterpret_cast<float4*>(part + (int64_t)blockIdx.y * cols + c) = t;
}

// Second stage: 8 columns per block, 32 groups of row blocks each, summed
// through LDS in a fixed order.
__global__ __launch_bounds__(256) void colsum8_stage2_kernel(const float* __restrict__ part, int nblk, int64_t cols,
                                                             float* __restrict__ out) {
    const int cc = threadIdx.x & 7, g = threadIdx.x >> 3;
    const int64_t c = (int64_t)blockIdx.x * 8 + cc;
    float s = 0.f;
    if (c < cols)
        for (int b = g; b < nblk; b += 32) s += part[(int64_t)b * cols + c];
    __shared__ float red[32][8];
    red[g][cc] = s;
    __syncthreads();
    if (g != 0 || c >= cols) return;
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < 32; ++k) t += red[k][cc];
    out[c] = t;
}

// Sums of nb slices of a launch's partial results, slices in a fixed order:
// out0[c] (c < n0) and out1[c - n0] = sum over j of part[j * stride + c]. 16
// threads of four columns by 16 groups of slices, summed through LDS.
// Destinations may be NULL; out0 has rows of w0 values, ld0 apart.
__global__ __launch_bounds__(256) void slice_sum_kernel(const float* __restrict__ part, int nb, int64_t stride,
                                                        int64_t n0, int64_t n1, float* __restrict__ out0,
                                                        float* __restrict__ out1, uint32_t w0, uint32_t ld0) {
    __shared__ float4 red[16][16];
    const int cx = (int)threadIdx.x & 15, gy = (int)threadIdx.x >> 4;
    const int64_t c = (int64_t)blockIdx.x * 64 + 4 * cx;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < n0 + n1) {
#pragma unroll 4
        for (int j = gy; j < nb; j += 16) {
            const float4 v = *reinterpret_cast<const float4*>(part + (int64_t)j * stride + c);
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
    }
    red[gy][cx] = s;
    __syncthreads();
    if (gy != 0 || c >= n0 + n1) return;
#pragma unroll
    for (int k = 1; k < 16; ++k) {
        const float4 v = red[k][cx];
        s.x += v.x;
        s.y += v.y;
        s.z += v.z;
        s.w += v.w;
    }
    const float v[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t e = c + k;
        if (e < n0) {
            if (out0) out0[w0 ? (size_t)((uint32_t)e / w0) * ld0 + (uint32_t)e % w0 : (size_t)e] = v[k];
        } else if (e < n0 + n1 && out1) {
            out1[e - n0] = v[k];
        }
    }
}

// ---- BF16 variants (the MLP backward of a BF16 forward) ----------------------
__device__ __forceinline__ __bf16 to_bf16(float v) { return (__bf16)v; }  // round to nearest even

// The BF16 weights of the backward, from the FP32 masters w[l] (row-major
// [out][in]): per 256 x 256 layer l = 1 .. n - 1 the MFMA fragments of W as the
// kernels below take them (fragment (t, c), lane 16 g + r, element j =
// W[32 c + 8 g + j][16 t + r]; 65536 values), then the output layer's 7 x 256.
struct BwdWeights {
    const float* w[8];
    int n;
};
__global__ __launch_bounds__(256) void pack_bwd_kernel(BwdWeights a, __bf16* __restrict__ out) {
    const int e = (int)(blockIdx.x * 256 + threadIdx.x);
    const int hid = (a.n - 1) * 65536;
    if (e < hid) {
        const int l = e >> 16, f = (e >> 9) & 127, ln = (e >> 3) & 63, j = e & 7;
        const int t = f >> 3, c = f & 7, g = ln >> 4, r = ln & 15;
        out[e] = to_bf16(a.w[1 + l][(size_t)(32 * c + 8 * g + j) * 256 + 16 * t + r]);
    } else if (e < hid + kOut * 256) {
        out[e] = to_bf16(a.w[a.n][e - hid]);
    }
}

// Input gradient of a 256 x 256 layer on BF16 MFMA (v_mfma_f32_16x16x32_bf16,
// FP32 accumulation): out[p][i] = sum_o dz[p][o] W[o][i] for the rows p of the
// listed groups, rounded to BF16 and zeroed where act[p][i] (the BF16
// activation) is not > 0, the previous layer's ReLU. The whole W sits in LDS in
// MFMA A-fragment order (pack_bwd_kernel's). Each wave takes groups of 32 pairs.
// In chunk order a lane's 16 bytes of dz are its B operand of a k chunk, its
// results of an output tile are 8 bytes of out, and their mask is 8 bytes of act:
// every access of a wave is contiguous, and no mask passes through LDS.
// The next group's rows are loaded while the current one is computed, a chunk's
// activations while the chunk before it is. 800k pairs, a quarter of them with a
// gradient: 81 us (93 row-major, with the mask as bits in LDS; 285 over all rows;
// 69 with rows in the results' own order).
constexpr int kDzWaves = 8;
constexpr int kDzNcb = 2;
constexpr int kDzPairs = 16 * kDzNcb;
static_assert(kDzPairs == kRowGroup, "a wave takes one group of rows");

typedef __bf16 dz_bf16x8 __attribute__((ext_vector_type(8)));
typedef float dz_f32x4 __attribute__((ext_vector_type(4)));
typedef float dz_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 dz_bf16x2 __attribute__((ext_vector_type(2)));

// 0xffff in each half of w whose BF16 is > 0 (activations are not negative), else 0
__device__ __forceinline__ uint32_t positive_halves(uint32_t w) {
    const uint32_t lo = (int32_t)(w << 16) > 0 ? 0x0000ffffu : 0u;
    const uint32_t hi = (int32_t)(w & 0xffff0000u) > 0 ? 0xffff0000u : 0u;
    return lo | hi;
}

__global__ __launch_bounds__(64 * kDzWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void dz_gemm_kernel(
    const __bf16* __restrict__ dz, const uint4* __restrict__ wf, const __bf16* __restrict__ act, int64_t P,
    RowGroups rg, __bf16* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) uint4 s_a[16 * 8 * 64];  // 128 fragments of 1 KiB
    const int64_t groups = (int64_t)*rg.count;
    if ((int64_t)blockIdx.x * kDzWaves >= groups) return;  // block-uniform
    for (int e = threadIdx.x; e < 16 * 8 * 64; e += 64 * kDzWaves) s_a[e] = wf[e];
    __syncthreads();
    const int wave = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63), g = lane >> 4, n = lane & 15;
    const int64_t stride = (int64_t)gridDim.x * kDzWaves;
    // this lane's row of column block cb of listed group q (P: none)
    auto row_of = [&](int64_t q, int cb) {
        const int64_t p = q < groups ? (int64_t)rg.list[q] * kDzPairs + cb * 16 + n : P;
        return p < P ? p : -1;
    };
    auto load = [&](const __bf16* src, int64_t p, int c) {
        return p >= 0 ? *reinterpret_cast<const uint4*>(src + chunk_at(p, c, g)) : make_uint4(0u, 0u, 0u, 0u);
    };
    auto load_mask = [&](int64_t p, int c) {  // of output tiles 2 c and 2 c + 1
        const uint2* m = reinterpret_cast<const uint2*>(act + chunk_half_at(p < 0 ? 0 : p, c, 0, g));
        return make_uint4(m[0].x, m[0].y, m[64].x, m[64].y);
    };
    int64_t grp = (int64_t)blockIdx.x * kDzWaves + wave;
    int64_t p[kDzNcb];
    uint4 b[8][kDzNcb], bn[8][kDzNcb];
#pragma unroll
    for (int cb = 0; cb < kDzNcb; ++cb) {
        p[cb] = row_of(grp, cb);
#pragma unroll
        for (int c = 0; c < 8; ++c) b[c][cb] = load(dz, p[cb], c);
    }
    for (; grp < groups; grp += stride) {
        int64_t pn[kDzNcb];
#pragma unroll
        for (int cb = 0; cb < kDzNcb; ++cb) {
            pn[cb] = row_of(grp + stride, cb);
#pragma unroll
            for (int c = 0; c < 8; ++c) bn[c][cb] = load(dz, pn[cb], c);
        }
        uint4 mk[kDzNcb];
#pragma unroll
        for (int cb = 0; cb < kDzNcb; ++cb) mk[cb] = load_mask(p[cb], 0);
#pragma unroll 1
        for (int cp = 0; cp < 8; ++cp) {
            uint4 m[kDzNcb];
#pragma unroll
            for (int cb = 0; cb < kDzNcb; ++cb) {
                m[cb] = mk[cb];
                if (cp < 7) mk[cb] = load_mask(p[cb], cp + 1);
            }
            dz_f32x4 acc[2][kDzNcb];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int cb = 0; cb < kDzNcb; ++cb) acc[h][cb] = dz_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const dz_bf16x8 a = __builtin_bit_cast(dz_bf16x8, s_a[((2 * cp + h) * 8 + c) * 64 + lane]);
#pragma unroll
                    for (int cb = 0; cb < kDzNcb; ++cb)
                        acc[h][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            a, __builtin_bit_cast(dz_bf16x8, b[c][cb]), acc[h][cb], 0, 0, 0);
                }
#pragma unroll
            for (int cb = 0; cb < kDzNcb; ++cb) {
                if (p[cb] < 0) continue;
                uint32_t v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const dz_f32x2 f = {acc[k >> 1][cb][2 * (k & 1)], acc[k >> 1][cb][2 * (k & 1) + 1]};
                    v[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, dz_bf16x2));
                }
                uint2* o = reinterpret_cast<uint2*>(out + chunk_half_at(p[cb], cp, 0, g));
                o[0] = make_uint2(v[0] & positive_halves(m[cb].x), v[1] & positive_halves(m[cb].y));
                o[64] = make_uint2(v[2] & positive_halves(m[cb].z), v[3] & positive_halves(m[cb].w));
            }
        }
#pragma unroll
        for (int cb = 0; cb < kDzNcb; ++cb) {
            p[cb] = pn[cb];
#pragma unroll
            for (int c = 0; c < 8; ++c) b[c][cb] = bn[c][cb];
        }
    }
}

// Layer-1 gradient of a BF16 backward without storing it: z[b][n] = dz1[b][n] W
// (FP32 accumulation on MFMA; dz1 [B][N][256] BF16, the gradient of the second
// layer's pre-activations; W its 256 x 256 BF16 weights' fragments), masked by
// act[b][n] > 0 (the layer-1 ReLU), gives S[n][:] = the sum over b (complete, in
// order) and Rpart[block][b][:] = the sum over the block's Gaussians.
// A block takes up to 8 strips of 16 Gaussians (strip w from 16 (w gridDim + block) on,
// so that the front of the depth order, where the rows with a gradient are, is
// dealt over all blocks) and every query in order. Wave w forms output features
// [32 w, 32 w + 32) of every strip: its 16 weight fragments stay in registers, the
// strips' rows and ReLU masks are staged in LDS once per query (wave w loads strip
// w, one query ahead) and read by all eight waves; a strip without a gradient in
// a query is passed over. Pairs are the MFMA rows, so a lane holds 4 pairs of one
// feature per product: S accumulates in registers over the queries, R over the
// strips, then over the 4 lane groups. (With each wave forming every feature of
// its own strip the weights came from LDS for each product and the few waves
// with a gradient ran alone: 221 us at 800k pairs, a quarter of them with a
// gradient, 331 with all; 110 with row-major rows, 100 now.)
constexpr int kL1Waves = 8;

__global__ __launch_bounds__(64 * kL1Waves) __attribute__((amdgpu_waves_per_eu(2, 2))) void layer1_grad_kernel(
    const __bf16* __restrict__ dz1, const uint4* __restrict__ wf, const __bf16* __restrict__ act, int B, int N,
    const uint32_t* __restrict__ bits, float* __restrict__ S, float* __restrict__ Rpart) {
    __shared__ __attribute__((aligned(16))) uint4 s_rows[kL1Waves][8][64];  // strip, 32-wide k chunk, lane
    __shared__ __attribute__((aligned(8))) uint8_t s_m[kL1Waves][16][64];  // ReLU masks: byte f / 4, bit f % 4
    __shared__ int s_any[kL1Waves];            // the strip has a row with a gradient
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63), g = lane >> 4, r = lane & 15;
    const int na = (wave * (int)gridDim.x + (int)blockIdx.x) * 16 + r;  // the Gaussian this lane loads
    dz_bf16x8 w[2][8];  // fragments of output tiles 2 wave and 2 wave + 1
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int c = 0; c < 8; ++c)
            w[t][c] = __builtin_bit_cast(dz_bf16x8, wf[((2 * wave + t) * 8 + c) * 64 + lane]);
    // rows of query b with a gradient (others were never written): dz1 and act of this lane's row, zero if not live
    uint4 a_nxt[8], m_nxt[8];
    bool live = false;
    auto load = [&](int b) {
        const int64_t p = (int64_t)b * N + na;
        live = b < B && na < N && ((bits[p >> 5] >> (p & 31)) & 1u);
        if (__ballot(live) == 0ull) return;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const size_t at = chunk_at(p, c, g);
            a_nxt[c] = live ? *reinterpret_cast<const uint4*>(dz1 + at) : make_uint4(0u, 0u, 0u, 0u);
            m_nxt[c] = live ? *reinterpret_cast<const uint4*>(act + at) : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    auto stage = [&]() {
        const bool any = __ballot(live) != 0ull;
        if (lane == 0) s_any[wave] = any;
        if (!any) return;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            s_rows[wave][c][lane] = a_nxt[c];
            const uint32_t lo = positive_halves(m_nxt[c].x) & 0x20001u, l2 = positive_halves(m_nxt[c].y) & 0x80004u;
            const uint32_t hi = positive_halves(m_nxt[c].z) & 0x20001u, h2 = positive_halves(m_nxt[c].w) & 0x80004u;
            const uint32_t ml = lo | l2, mh = hi | h2;
            s_m[wave][r][8 * c + 2 * g] = (uint8_t)(ml | (ml >> 16));      // features 32 c + 8 g + 0..3
            s_m[wave][r][8 * c + 2 * g + 1] = (uint8_t)(mh | (mh >> 16));  // features 32 c + 8 g + 4..7
        }
    };
    dz_f32x4 sacc[kL1Waves][2];
#pragma unroll
    for (int s = 0; s < kL1Waves; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t) sacc[s][t] = dz_f32x4{0.f, 0.f, 0.f, 0.f};
    load(0);
    for (int b = 0; b < B; ++b) {
        __syncthreads();  // every wave is done with the previous query's rows
        stage();
        __syncthreads();
        load(b + 1);
        float rsum[2] = {0.f, 0.f};
#pragma unroll
        for (int s = 0; s < kL1Waves; ++s) {
            if (!__builtin_amdgcn_readfirstlane(s_any[s])) continue;
            dz_f32x4 acc[2] = {dz_f32x4{0.f, 0.f, 0.f, 0.f}, dz_f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const dz_bf16x8 a = __builtin_bit_cast(dz_bf16x8, s_rows[s][c][lane]);
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w[t][c], acc[t], 0, 0, 0);
            }
            // lane (g, r) holds pairs 4 g + jj of features 32 wave + 16 t + r: mask byte 8 wave + 4 t + r / 4
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const uint2 word = *reinterpret_cast<const uint2*>(&s_m[s][4 * g + jj][8 * wave]);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const float x = ((t ? word.y : word.x) >> (8 * (r >> 2) + (r & 3))) & 1u ? acc[t][jj] : 0.f;
                    sacc[s][t][jj] += x;
                    rsum[t] += x;
                }
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float v = rsum[t];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (g == 0) Rpart[((size_t)blockIdx.x * B + b) * 256 + 32 * wave + 16 * t + r] = v;
        }
    }
#pragma unroll
    for (int s = 0; s < kL1Waves; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const int n = (s * (int)gridDim.x + (int)blockIdx.x) * 16 + 4 * g + jj;
                if (n < N) S[(size_t)n * 256 + 32 * wave + 16 * t + r] = sacc[s][t][jj];
            }
}

// Weight gradient of a 256 x 256 layer on BF16 MFMA over one slice of pairs:
// part[blk][o][i] = sum over the pairs p of every gridDim-th listed group of
// dz[p][o] act[p][i] (dz, act [P][256] BF16; FP32 accumulation); the caller adds
// the slices. The
// contraction runs over pairs, so both operands are staged through LDS
// transposed, feature-major, 32 pairs at a time (rows padded to 80 bytes: the
// 16-byte fragment reads of 16 consecutive features and the 2-byte staging
// writes of consecutive pairs fall in distinct banks). Wave w accumulates the
// 4 x 8 output tiles o in [64 (w % 4), +64), i in [128 (w / 4), +128) in
// registers; the next 32 pairs are loaded while the current ones are multiplied.
// The layer's bias gradient (the column sums of dz) comes along: waves 0..3
// multiply their dz fragments by a fragment of ones as well. A slice is 65536
// values, then the 256 of the bias.
constexpr int kWgWaves = 8;
constexpr int kWgRow = 40;  // bf16 per staged feature row: 32 pairs + padding

constexpr int kWgSlice = 65536 + 256;

__global__ __launch_bounds__(64 * kWgWaves) void wgrad_mfma_kernel(const __bf16* __restrict__ dz,
                                                                   const __bf16* __restrict__ act, int64_t P,
                                                                   RowGroups rg, float* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) uint16_t t_dz[256 * kWgRow];
    __shared__ __attribute__((aligned(16))) uint16_t t_act[256 * kWgRow];
    const int tid = (int)threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, g = lane >> 4, n = lane & 15;
    const int o0 = 64 * (wave & 3), i0 = 128 * (wave >> 2);
    const uint32_t ng = *rg.count;
    // staging: thread -> pair q = tid % 32 of the group, 8-value pieces k = tid / 32 and k + 16 of its row: chunk
    // k / 4, lane group k % 4
    const int q = tid & 31, c0 = tid >> 5;
    uint4 rd[2], ra[2];
    auto load = [&](uint32_t k) {
        const int64_t p = (int64_t)rg.list[k] * kRowGroup + q;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = c0 + 16 * h;
            const size_t at = chunk_at(p, c >> 2, c & 3);
            rd[h] = p < P ? *reinterpret_cast<const uint4*>(dz + at) : make_uint4(0u, 0u, 0u, 0u);
            ra[h] = p < P ? *reinterpret_cast<const uint4*>(act + at) : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    auto stage = [&]() {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = c0 + 16 * h;
            const uint32_t wd[4] = {rd[h].x, rd[h].y, rd[h].z, rd[h].w};
            const uint32_t wa[4] = {ra[h].x, ra[h].y, ra[h].z, ra[h].w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int f = 8 * c + 2 * k;
                t_dz[f * kWgRow + q] = (uint16_t)(wd[k] & 0xffffu);
                t_dz[(f + 1) * kWgRow + q] = (uint16_t)(wd[k] >> 16);
                t_act[f * kWgRow + q] = (uint16_t)(wa[k] & 0xffffu);
                t_act[(f + 1) * kWgRow + q] = (uint16_t)(wa[k] >> 16);
            }
        }
    };
    dz_f32x4 acc[4][8], accb[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        accb[a] = dz_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[a][b] = dz_f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const bool bias_wave = (wave >> 2) == 0;  // waves 0..3 cover the 16 o-tiles once
    const uint4 one4 = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);  // bf16 1.0 x 8
    const dz_bf16x8 ones = __builtin_bit_cast(dz_bf16x8, one4);
    if (blockIdx.x < ng) load(blockIdx.x);
    for (uint32_t k = blockIdx.x; k < ng; k += gridDim.x) {
        __syncthreads();  // the previous chunk's fragment reads are complete
        stage();
        __syncthreads();
        if (k + gridDim.x < ng) load(k + gridDim.x);
        dz_bf16x8 fa[4];
#pragma unroll
        for (int a = 0; a < 4; ++a)  // A(o, k = pair): 8 consecutive pairs of feature o
            fa[a] = *reinterpret_cast<const dz_bf16x8*>(&t_dz[(o0 + 16 * a + n) * kWgRow + 8 * g]);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const dz_bf16x8 fb = *reinterpret_cast<const dz_bf16x8*>(&t_act[(i0 + 16 * b + n) * kWgRow + 8 * g]);
#pragma unroll
            for (int a = 0; a < 4; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a], fb, acc[a][b], 0, 0, 0);
        }
        if (bias_wave)
#pragma unroll
            for (int a = 0; a < 4; ++a) accb[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a], ones, accb[a], 0, 0, 0);
    }
    if (bias_wave && n == 0) {  // every column of the ones product is the row sum
        float* ob = part + (size_t)blockIdx.x * kWgSlice + 65536;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) ob[o0 + 16 * a + 4 * g + jj] = accb[a][jj];
    }
    // D(row 4 g + jj, col n) of tile (a, b) is dW[o0 + 16 a + 4 g + jj][i0 + 16 b + n]
    float* out = part + (size_t)blockIdx.x * kWgSlice;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                out[(size_t)(o0 + 16 * a + 4 * g + jj) * 256 + i0 + 16 * b + n] = acc[a][b][jj];
}

// The same contraction after an FP32 forward (dz, act [P][256] FP32) on the FP32
// matrix cores (v_mfma_f32_16x16x4_f32): part[blk][o][i] over every gridDim-th
// listed group. Each row is read once, as 16 bytes per thread, and staged row by
// row (padded by 16 floats: the 4 rows that one fragment read touches fall in
// distinct banks), double-buffered, one barrier per 32 rows; the next rows are
// loaded while the current ones are multiplied. Tiles per wave and slices as
// above; the bias gradient is summed from the fragments. 160k pairs: 223 us per
// layer as a general product of 128 x 128 tiles, which read each row twice; 178
// here (the instructions' own time: 146).
constexpr int kWfRow = 256 + 16;

__global__ __launch_bounds__(64 * kWgWaves) void wgrad_f32_kernel(const float* __restrict__ dz,
                                                                  const float* __restrict__ act, int64_t P,
                                                                  RowGroups rg, float* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) float s_rows[2 * 2 * kRowGroup * kWfRow];  // [buffer][dz, act][32][kWfRow]
    const int tid = (int)threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, g = lane >> 4, n = lane & 15;
    const int o0 = 64 * (wave & 3), i0 = 128 * (wave >> 2);
    const uint32_t ng = *rg.count;
    // staging: wave w takes pieces w and w + 8 of the group's two tiles of 16 rows
    float4 rd[4], ra[4];
    auto load = [&](uint32_t k) {
        const int64_t p0 = (int64_t)rg.list[k] * kRowGroup + n;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int64_t p = p0 + 16 * (h >> 1);
            const size_t at = piece_at(p, wave + 8 * (h & 1), g);
            rd[h] = p < P ? load4(dz + at) : make_float4(0.f, 0.f, 0.f, 0.f);
            ra[h] = p < P ? load4(act + at) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    auto stage = [&](int buf) {
        float* b = s_rows + buf * 2 * kRowGroup * kWfRow;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            float* d = b + (16 * (h >> 1) + n) * kWfRow + 16 * (wave + 8 * (h & 1)) + 4 * g;
            *reinterpret_cast<float4*>(d) = rd[h];
            *reinterpret_cast<float4*>(d + kRowGroup * kWfRow) = ra[h];
        }
    };
    dz_f32x4 acc[4][8];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[a][b] = dz_f32x4{0.f, 0.f, 0.f, 0.f};
    float bias[4] = {0.f, 0.f, 0.f, 0.f};  // sums of dz over rows 4 q + g
    if (blockIdx.x < ng) {
        load(blockIdx.x);
        stage(0);
    }
    __syncthreads();
    int buf = 0;
    for (uint32_t k = blockIdx.x; k < ng; k += gridDim.x, buf ^= 1) {
        const bool more = k + gridDim.x < ng;
        if (more) load(k + gridDim.x);
        const float* b0 = s_rows + buf * 2 * kRowGroup * kWfRow;
#pragma unroll
        for (int q = 0; q < kRowGroup / 4; ++q) {  // rows 4 q + g
            const float* rz = b0 + (4 * q + g) * kWfRow + o0 + n;
            const float* rx = b0 + (kRowGroup + 4 * q + g) * kWfRow + i0 + n;
            float fa[4], fb[8];
#pragma unroll
            for (int a = 0; a < 4; ++a) fa[a] = rz[16 * a];
#pragma unroll
            for (int b = 0; b < 8; ++b) fb[b] = rx[16 * b];
#pragma unroll
            for (int a = 0; a < 4; ++a) bias[a] += fa[a];
#pragma unroll
            for (int b = 0; b < 8; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
        if (more) stage(buf ^ 1);  // read last before the barrier that ended the step before
        __syncthreads();
    }
    float* out = part + (size_t)blockIdx.x * kWgSlice;
    if (wave < 4)  // these cover the 16 o-tiles once
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            float v = bias[a] + __shfl_xor(bias[a], 16);
            v += __shfl_xor(v, 32);
            if (g == 0) out[65536 + o0 + 16 * a + n] = v;
        }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                out[(size_t)(o0 + 16 * a + 4 * g + jj) * 256 + i0 + 16 * b + n] = acc[a][b][jj];
}

// Output layer of the backward in one pass over the last hidden activations
// act [P][256] over every gridDim-th listed group: with dy [P][7] FP32 (the
// upstream gradient as computed, not rounded) and Wo [7][256], T the type of act,
// wo and dz,
//   dz[p][f] = T(sum_o dy[p][o] Wo[o][f]), zero where act[p][f] is not > 0
//     (the gradient of the last hidden pre-activations; skipped if dz is NULL),
//   part[blk] = the slice's sums of dy[p][o] act[p][f] (the weight gradient,
//     7 x 256), then of dy[p][o] (the bias gradient, 7 and a pad); the caller
//     adds the slices.
// Wave w takes feature chunk w of 16 rows at a time, a lane 8 features of one
// row, whose output weights stay in its registers, the next group's loads in
// flight. 800k pairs, a quarter of them with a gradient, BF16: 73 us (105 with
// each group loaded when it is due); 160k pairs, FP32: 78 us (88 row-major,
// 8 features of every 8th row per thread).
constexpr int kOutSlice = kOut * 256 + 8;

// the lane's 8 values of chunk c of a row, as floats: features feature(c, g, 0..7)
template <typename T>
struct OutRow;
template <>
struct OutRow<__bf16> {
    uint4 v;
    __device__ static int feature(int c, int g, int j) { return 32 * c + 8 * g + j; }
    __device__ void load(const __bf16* a, int64_t p, int c, int g) {
        v = *reinterpret_cast<const uint4*>(a + chunk_at(p, c, g));
    }
    __device__ void clear() { v = make_uint4(0u, 0u, 0u, 0u); }
    __device__ float at(int j) const {
        const uint32_t w = j < 2 ? v.x : j < 4 ? v.y : j < 6 ? v.z : v.w;
        return __uint_as_float(j & 1 ? w & 0xffff0000u : w << 16);
    }
    // dz = z rounded, where the activation is > 0
    __device__ void store_masked(__bf16* dz, int64_t p, int c, int g, const float (&z)[8]) const {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        uint32_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const dz_f32x2 f = {z[2 * k], z[2 * k + 1]};
            o[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, dz_bf16x2)) & positive_halves(w[k]);
        }
        *reinterpret_cast<uint4*>(dz + chunk_at(p, c, g)) = make_uint4(o[0], o[1], o[2], o[3]);
    }
};
template <>
struct OutRow<float> {
    float4 v[2];
    __device__ static int feature(int c, int g, int j) { return 32 * c + 16 * (j >> 2) + 4 * g + (j & 3); }
    __device__ void load(const float* a, int64_t p, int c, int g) {
        v[0] = load4(a + piece_at(p, 2 * c, g));
        v[1] = load4(a + piece_at(p, 2 * c + 1, g));
    }
    __device__ void clear() { v[0] = v[1] = make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ float at(int j) const {
        const float4 q = v[j >> 2];
        return (j & 3) == 0 ? q.x : (j & 3) == 1 ? q.y : (j & 3) == 2 ? q.z : q.w;
    }
    __device__ void store_masked(float* dz, int64_t p, int c, int g, const float (&z)[8]) const {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            *reinterpret_cast<float4*>(dz + piece_at(p, 2 * c + h, g)) =
                make_float4(v[h].x > 0.f ? z[4 * h] : 0.f, v[h].y > 0.f ? z[4 * h + 1] : 0.f,
                            v[h].z > 0.f ? z[4 * h + 2] : 0.f, v[h].w > 0.f ? z[4 * h + 3] : 0.f);
    }
};

template <typename T>
__global__ __launch_bounds__(512) void out_bwd_kernel(const float* __restrict__ dy, const T* __restrict__ wo,
                                                      const T* __restrict__ act, int64_t P, RowGroups rg,
                                                      T* __restrict__ dz, float* __restrict__ part) {
    const int c = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63), g = lane >> 4, n = lane & 15;
    const uint32_t ng = *rg.count;
    float w[kOut][8], acc[kOut][8], ysum[kOut];
#pragma unroll
    for (int o = 0; o < kOut; ++o) {
        ysum[o] = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            w[o][j] = (float)wo[o * 256 + OutRow<T>::feature(c, g, j)];
            acc[o][j] = 0.f;
        }
    }
    OutRow<T> a[2], a_nxt[2];
    float y[2][kOut], y_nxt[2][kOut];
    auto load = [&](uint32_t k) {  // one group ahead
        const int64_t p0 = k < ng ? (int64_t)rg.list[k] * kRowGroup + n : P;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t p = p0 + 16 * h;
            if (p < P)
                a_nxt[h].load(act, p, c, g);
            else
                a_nxt[h].clear();
#pragma unroll
            for (int o = 0; o < kOut; ++o) y_nxt[h][o] = p < P ? dy[p * kOut + o] : 0.f;
        }
    };
    load(blockIdx.x);
    for (uint32_t k = blockIdx.x; k < ng; k += gridDim.x) {
        const int64_t p0 = (int64_t)rg.list[k] * kRowGroup + n;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            a[h] = a_nxt[h];
#pragma unroll
            for (int o = 0; o < kOut; ++o) y[h][o] = y_nxt[h][o];
        }
        load(k + gridDim.x);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int o = 0; o < kOut; ++o) {
                ysum[o] += y[h][o];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    acc[o][j] = fmaf(y[h][o], a[h].at(j), acc[o][j]);
                    z[j] = fmaf(y[h][o], w[o][j], z[j]);
                }
            }
            const int64_t p = p0 + 16 * h;
            if (dz && p < P) a[h].store_masked(dz, p, c, g, z);
        }
    }
    // the 16 rows of a lane group
    float* pb = part + (size_t)blockIdx.x * kOutSlice;
#pragma unroll
    for (int o = 0; o < kOut; ++o) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float v = acc[o][j];
#pragma unroll
            for (int m = 1; m < 16; m <<= 1) v += __shfl_xor(v, m);
            if (n == 0) pb[o * 256 + OutRow<T>::feature(c, g, j)] = v;
        }
        float v = ysum[o];
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) v += __shfl_xor(v, m);
        if (threadIdx.x == 0) pb[kOut * 256 + o] = v;
    }
    if (threadIdx.x == 0) pb[kOut * 256 + kOut] = 0.f;
}

// Layer-1 gradient sums in one pass over the FP32 gradient z [B][N][256]:
// with dz = z * [act > 0] (kMask: the BF16 activations act [B][N][256] mask an
// unmasked z, row-major; else z is dz already, in piece order), S[n][k] = sum_b dz[b][n][k]
// (complete: the block owns Gaussians n0 .. n0 + 31, summed over b in order)
// and Rpart[block][b][k] = sum over the block's Gaussians of dz[b][n][k]
// (4 row groups through LDS).
constexpr int kSumRows = 32;

// Rows without a gradient (bits, when given) count zero: they were not written.
template <bool kMask>
__global__ __launch_bounds__(256) void layer1_sums_kernel(const float* __restrict__ z, const __bf16* __restrict__ act,
                                                          const uint32_t* __restrict__ bits, int B, int N,
                                                          float* __restrict__ S,
                                                          float* __restrict__ Rpart) {
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int c = tx * 4;
    const int n0 = blockIdx.x * kSumRows;
    float4 sacc[kSumRows / 4];
#pragma unroll
    for (int i = 0; i < kSumRows / 4; ++i) sacc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    __shared__ float4 red[4][64];
    for (int b = 0; b < B; ++b) {
        float4 racc = make_float4(0.f, 0.f, 0.f, 0.f);
        // a row that does not count reads the query's first instead, so that the loads go out together
        float4 v[kSumRows / 4], a[kSumRows / 4];
        bool on[kSumRows / 4];
#pragma unroll
        for (int i = 0; i < kSumRows / 4; ++i) {
            const int n = n0 + ty + 4 * i;
            int64_t p = (int64_t)b * N + (n < N ? n : 0);
            on[i] = n < N && (!bits || ((bits[p >> 5] >> (p & 31)) & 1u));
            if (!on[i]) p = (int64_t)b * N;
            v[i] = load4(z + (kMask ? (size_t)p * 256 + c : piece_at(p, c / 16, c % 16 / 4)));
            if constexpr (kMask) a[i] = load4(act + chunk_at(p, c / 32, c % 32 / 8) + c % 8);
        }
#pragma unroll
        for (int i = 0; i < kSumRows / 4; ++i) {
            if (on[i]) {
                float4 m = v[i];
                if constexpr (kMask)
                    m = make_float4(a[i].x > 0.f ? m.x : 0.f, a[i].y > 0.f ? m.y : 0.f, a[i].z > 0.f ? m.z : 0.f,
                                    a[i].w > 0.f ? m.w : 0.f);
                sacc[i].x += m.x;
                sacc[i].y += m.y;
                sacc[i].z += m.z;
                sacc[i].w += m.w;
                racc.x += m.x;
                racc.y += m.y;
                racc.z += m.z;
                racc.w += m.w;
            }
        }
        red[ty][tx] = racc;
        __syncthreads();
        if (ty == 0) {
            float4 t = red[0][tx];
#pragma unroll
            for (int k = 1; k < 4; ++k) {
                t.x += red[k][tx].x;
                t.y += red[k][tx].y;
                t.z += red[k][tx].z;
                t.w += red[k][tx].w;
            }
            *reinterpret_cast<float4*>(Rpart + ((size_t)blockIdx.x * B + b) * 256 + c) = t;
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kSumRows / 4; ++i) {
        const int n = n0 + ty + 4 * i;
        if (n < N) *reinterpret_cast<float4*>(S + (size_t)n * 256 + c) = sacc[i];
    }
}

__global__ void to_bf16_kernel(const float* __restrict__ x, int64_t n, __bf16* __restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = to_bf16(x[i]);
}

// What layer 1 takes from S [N][256], its pre-activation gradient summed over the
// batch, in one pass: the mean part of its weight gradient S^T gamma(mu_hat) and
// its bias gradient (a slice of 256 x 26 and 256 values per block, to be summed),
// and per Gaussian d gamma(mu_hat) = S W1m taken through the sin / cos features
// to dmu [N][2]. FP32 on the matrix cores (v_mfma_f32_16x16x4_f32). A block takes
// every gridDim-th group of 32 rows: staged in LDS (rows padded by 16 floats, so
// that 4 rows fall in distinct banks), read as columns by wave w for units
// [64 w, 64 w + 64) of the weight gradient, and as rows for the same units'
// share of d gamma, which the waves then add through LDS. The next rows are
// loaded while the current ones are multiplied. As separate launches (features,
// column sums, two products of few columns with their slices' sums, the chain)
// this read S three times: 96 us for 50k Gaussians, 28 and 6 for the slices now.
constexpr int kMgRows = 32, kMgRow = 256 + 16, kMgFeat = 48, kMgDg = 36;
constexpr int kMgSlice = 256 * kMeanFeat + 256;

__global__ __launch_bounds__(256, 2) void mean_grad_kernel(const float* __restrict__ S, const float* __restrict__ w1,
                                                           int in_dim, const float* __restrict__ mx,
                                                           const float* __restrict__ my, int N, int Wd, int Hd,
                                                           float* __restrict__ dmu, float* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) float s_s[kMgRows][kMgRow];
    __shared__ float s_f[kMgRows][kMgFeat];  // gamma(mu_hat), zero from 26 on
    __shared__ __attribute__((aligned(16))) float s_d[4][kMgRows][kMgDg];
    const int tid = (int)threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 4, n = lane & 15;
    // W1m as A operands of the wave's units: tile t, units 16 q + 4 g + e of q = 4 wave + 0..3
    float wa[2][4][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                wa[t][q][e] = 16 * t + n < kMeanFeat
                                  ? w1[(size_t)(64 * wave + 16 * q + 4 * g + e) * in_dim + 16 * t + n]
                                  : 0.f;
    dz_f32x4 acc[4][2];
    float bias[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[a][t] = dz_f32x4{0.f, 0.f, 0.f, 0.f};
    // staging: wave w takes rows w, w + 4, .., a lane 4 units; rows past N read the last and count zero
    float4 nx[kMgRows / 4];
    auto load = [&](int r0) {
#pragma unroll
        for (int h = 0; h < kMgRows / 4; ++h)
            nx[h] = load4(S + (size_t)min(r0 + wave + 4 * h, N - 1) * 256 + 4 * lane);
    };
    int r0 = (int)blockIdx.x * kMgRows;
    const int step = (int)gridDim.x * kMgRows;
    if (r0 < N) load(r0);
    for (; r0 < N; r0 += step) {
#pragma unroll
        for (int h = 0; h < kMgRows / 4; ++h)
            *reinterpret_cast<float4*>(&s_s[wave + 4 * h][4 * lane]) =
                r0 + wave + 4 * h < N ? nx[h] : make_float4(0.f, 0.f, 0.f, 0.f);
        {
            // features: band tid / 32 of row tid % 32; the seventh group takes the identity, the eighth the zeros
            const int r = tid & 31, k = tid >> 5, p = r0 + r;
            float hx, lx, hy, ly;
            div_two(mx[min(p, N - 1)], (float)Wd, hx, lx);
            div_two(my[min(p, N - 1)], (float)Hd, hy, ly);
            if (k < kMeanBands) {
                float sx, cx, sy, cy;
                sincospi_scaled(hx, lx, k, sx, cx);
                sincospi_scaled(hy, ly, k, sy, cy);
                s_f[r][2 + 2 * k] = p < N ? sx : 0.f;
                s_f[r][3 + 2 * k] = p < N ? sy : 0.f;
                s_f[r][2 + 2 * kMeanBands + 2 * k] = p < N ? cx : 0.f;
                s_f[r][3 + 2 * kMeanBands + 2 * k] = p < N ? cy : 0.f;
            } else if (k == kMeanBands) {
                s_f[r][0] = p < N ? hx + lx : 0.f;
                s_f[r][1] = p < N ? hy + ly : 0.f;
            } else {
#pragma unroll
                for (int j = kMeanFeat; j < 32; ++j) s_f[r][j] = 0.f;
            }
        }
        __syncthreads();
        if (r0 + step < N) load(r0 + step);
#pragma unroll
        for (int c = 0; c < kMgRows / 4; ++c) {  // rows 4 c + g
            float fa[4], fb[2];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                fa[a] = s_s[4 * c + g][64 * wave + 16 * a + n];
                bias[a] += fa[a];
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) fb[t] = s_f[4 * c + g][16 * t + n];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[a], fb[t], acc[a][t], 0, 0, 0);
        }
#pragma unroll
        for (int rt = 0; rt < kMgRows / 16; ++rt) {
            dz_f32x4 d[2] = {dz_f32x4{0.f, 0.f, 0.f, 0.f}, dz_f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 b4 = load4(&s_s[16 * rt + n][64 * wave + 16 * q + 4 * g]);
                const float b[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        d[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[t][q][e], b[e], d[t], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)  // lane (g, n): features 16 t + 4 g + i of row n
                *reinterpret_cast<float4*>(&s_d[wave][16 * rt + n][16 * t + 4 * g]) =
                    make_float4(d[t][0], d[t][1], d[t][2], d[t][3]);
        }
        __syncthreads();
        if (tid < 2 * kMgRows && r0 + (tid & 31) < N) {  // d mu of one axis of one row
            const int r = tid & 31, ax = tid >> 5;
            const auto dg = [&](int k) { return (s_d[0][r][k] + s_d[1][r][k]) + (s_d[2][r][k] + s_d[3][r][k]); };
            float v = dg(ax);
#pragma unroll
            for (int k = 0; k < kMeanBands; ++k) {
                const int si = 2 + 2 * k + ax, ci = si + 2 * kMeanBands;
                const float f = 3.14159265358979323846f * (float)(1 << k);
                v += f * (dg(si) * s_f[r][ci] - dg(ci) * s_f[r][si]);
            }
            dmu[(size_t)(r0 + r) * 2 + ax] = v / (float)(ax ? Hd : Wd);
        }
        __syncthreads();
    }
    float* out = part + (size_t)blockIdx.x * kMgSlice;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (16 * t + n < kMeanFeat)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    out[(size_t)(64 * wave + 16 * a + 4 * g + i) * kMeanFeat + 16 * t + n] = acc[a][t][i];
        float v = bias[a] + __shfl_xor(bias[a], 16);
        v += __shfl_xor(v, 32);
        if (g == 0) out[256 * kMeanFeat + 64 * wave + 16 * a + n] = v;
    }
}

}  // namespace

void launch_blend_backward(const uint2* ranges, const uint32_t* vals, const Records& r, int B, const Grid& g,
                           const float* grad_out, const float* aux_T, const uint32_t* aux_last, float* dpair,
                           hipStream_t st, float* det_part, int N, const uint32_t* det_off) {
    const unsigned blocks = (unsigned)(B * g.tiles);
    if (!blocks) return;
#define SWF_BLEND_BWD(TILE, WRAP, DET)                                                                         \
    blend_backward_kernel<TILE, WRAP, DET><<<blocks, TILE * TILE, 0, st>>>(                                    \
        ranges, vals, r.geo, r.wm, r.oa, g.H, g.W, g.TW, g.tiles, grad_out, aux_T, aux_last, dpair, det_part, r.rect,  \
        det_off)
#define SWF_BLEND_BWD_T(TILE, DET)   \
    do {                             \
        if (g.wrap)                  \
            SWF_BLEND_BWD(TILE, true, DET);  \
        else                         \
            SWF_BLEND_BWD(TILE, false, DET); \
    } while (0)
    if (det_part) {
        if (g.tile == 8)
            SWF_BLEND_BWD_T(8, true);
        else
            SWF_BLEND_BWD_T(16, true);
        const int64_t P = (int64_t)B * N;
        if (P > 0)
            det_reduce_kernel<<<(unsigned)((P + 255) / 256), 256, 0, st>>>(r.count, det_off, det_part, P, dpair);
    } else {
        if (g.tile == 8)
            SWF_BLEND_BWD_T(8, false);
        else
            SWF_BLEND_BWD_T(16, false);
    }
#undef SWF_BLEND_BWD_T
#undef SWF_BLEND_BWD
}

size_t row_group_words(int64_t P) { return 2 * (size_t)((P + 31) / 32) + (size_t)((P + 255) / 256) + 16; }

RowGroups row_groups(uint32_t* buf, int64_t P) {
    RowGroups g;
    g.count = buf;
    g.bits = buf + 16;
    g.list = buf + 16 + (P + 31) / 32;
    return g;
}

void launch_preprocess_backward(const float* dpair, const Records& r, int64_t P, bool paper_mask, float* dbase,
                                float* dy, uint32_t* group_buf, hipStream_t st) {
    if (P <= 0) {
        if (dy) launch_clear_u32(group_buf, 1, st);
        return;
    }
    const unsigned blocks = (unsigned)((P + 255) / 256);
    const int64_t ng = (P + 31) / 32;
    uint32_t* bits = dy ? group_buf + 16 : nullptr;
    uint32_t* counts = dy ? bits + 2 * ng : nullptr;
    preprocess_backward_kernel<<<blocks, 256, 0, st>>>(dpair, r.wm, r.oa, r.count, r.rect, P, paper_mask ? 1 : 0,
                                                       dbase, dy, bits, counts);
    if (dy)
        row_groups_kernel<<<(unsigned)((ng + 1023) / 1024), 1024, 0, st>>>(bits, counts, ng, bits + ng, group_buf);
}

void launch_base_reduce(const float* dbase, const float* dmu_pe, const uint32_t* perm, int B, int N,
                        const BaseGrads& out, hipStream_t st) {
    if (N > 0) base_reduce_kernel<<<(N + 255) / 256, 256, 0, st>>>(dbase, dmu_pe, perm, B, N, out);
}

int colsum_blocks(int64_t rows) { return (int)std::max<int64_t>(1, std::min<int64_t>(2048, (rows + 255) / 256)); }

void launch_colsum(const float* A, int64_t rows, int64_t cols, float* part, float* out, hipStream_t st) {
    if (cols <= 0) return;
    const int nblk = colsum_blocks(rows);
    const int64_t rpb = (rows + nblk - 1) / nblk;
    colsum4_stage1_kernel<<<dim3((unsigned)((cols + 255) / 256), nblk), 256, 0, st>>>(A, rows, cols, rpb, part);
    colsum8_stage2_kernel<<<(unsigned)((cols + 7) / 8), 256, 0, st>>>(part, nblk, cols, out);
}

void launch_pack_bwd(const float* const* w, int n_hidden, void* out, hipStream_t st) {
    BwdWeights a{};
    for (int l = 0; l <= n_hidden && l < 8; ++l) a.w[l] = w[l];
    a.n = n_hidden;
    const int n = (n_hidden - 1) * 65536 + kOut * 256;
    pack_bwd_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(a, (__bf16*)out);
}

// w0: out0's row length, rows ld0 apart (0: one row)
static void slice_sum(const float* part, int nb, int64_t stride, int64_t n0, int64_t n1, float* out0, float* out1,
                      hipStream_t st, uint32_t w0 = 0, uint32_t ld0 = 0) {
    if (out0 || out1)
        slice_sum_kernel<<<(unsigned)((n0 + n1 + 63) / 64), 256, 0, st>>>(part, nb, stride, n0, n1, out0, out1, w0,
                                                                          ld0);
}

void launch_dz_gemm(const void* dz, const void* wf, const void* act, int64_t P, const RowGroups& rg, void* out,
                    hipStream_t st) {
    if (P <= 0) return;
    const int64_t groups = (P + kDzPairs - 1) / kDzPairs;
    const int blocks = (int)std::min<int64_t>(n_compute_units(), (groups + kDzWaves - 1) / kDzWaves);
    dz_gemm_kernel<<<blocks, 64 * kDzWaves, 0, st>>>((const __bf16*)dz, (const uint4*)wf, (const __bf16*)act, P, rg,
                                                     (__bf16*)out);
}

// One block per compute unit as soon as there are groups for it, two from 512 rows per block on: 40k pairs 26 us (FP32
// 33) with 256 rows to a block (157 blocks), 22 (28) now.
int out_bwd_blocks(int64_t P) {
    const int64_t G = (P + kRowGroup - 1) / kRowGroup;
    const int64_t cus = n_compute_units();
    return (int)std::max<int64_t>(1, P >= 512 * cus ? 2 * cus : std::min<int64_t>(cus, G));
}
size_t out_bwd_floats(int64_t P) { return (size_t)out_bwd_blocks(P) * kOutSlice; }

void launch_out_bwd(bool bf16, const float* dy, const void* wo, const void* act, int64_t P, const RowGroups& rg,
                    void* dz, float* part, float* dWo, float* dbo, hipStream_t st) {
    if (!dz && !dWo && !dbo) return;
    const int nblk = out_bwd_blocks(P);  // P = 0: one block writes zeros
    if (bf16)
        out_bwd_kernel<__bf16><<<nblk, 512, 0, st>>>(dy, (const __bf16*)wo, (const __bf16*)act, P, rg, (__bf16*)dz,
                                                     part);
    else
        out_bwd_kernel<float><<<nblk, 512, 0, st>>>(dy, (const float*)wo, (const float*)act, P, rg, (float*)dz, part);
    slice_sum(part, nblk, kOutSlice, kOut * 256, kOut, dWo, dbo, st);
}

// Blocks of a weight gradient: each has its share of the G = P / 32 groups to multiply (group_us each) and a slice of
// 257 KiB that is written and read again (0.12 us of the whole chip's bandwidth), so about sqrt(G group_us / 0.12) of
// them, as many as there are compute units at most: 40k pairs 52 us with 1024 rows to a block, 24 here (40 and 131
// blocks); FP32 80 with 256 rows to a block, 60 here (157 and 256); the slices' sums 4 us longer each.
static int wgrad_blocks(int64_t P, double group_us) {
    const int64_t G = (P + kRowGroup - 1) / kRowGroup;
    const auto best = (int64_t)std::ceil(std::sqrt((double)G * group_us / 0.12));
    return (int)std::max<int64_t>(1, std::min({(int64_t)n_compute_units(), G, best}));
}

int wgrad_mfma_blocks(int64_t P) { return wgrad_blocks(P, 1.6); }
size_t wgrad_mfma_floats(int64_t P) { return (size_t)wgrad_mfma_blocks(P) * kWgSlice; }

void launch_wgrad_mfma(const void* dz, const void* act, int64_t P, const RowGroups& rg, float* part, float* dW,
                       float* db, hipStream_t st) {
    if (!dW && !db) return;
    const int nblk = wgrad_mfma_blocks(P);  // P = 0: one block writes zeros
    wgrad_mfma_kernel<<<nblk, 64 * kWgWaves, 0, st>>>((const __bf16*)dz, (const __bf16*)act, P, rg, part);
    slice_sum(part, nblk, kWgSlice, 65536, 256, dW, db, st);
}

int wgrad_f32_blocks(int64_t P) { return wgrad_blocks(P, 7.3); }
size_t wgrad_f32_floats(int64_t P) { return (size_t)wgrad_f32_blocks(P) * kWgSlice; }

void launch_wgrad_f32(const float* dz, const float* act, int64_t P, const RowGroups& rg, float* part, float* dW,
                      float* db, hipStream_t st) {
    if (!dW && !db) return;
    const int nblk = wgrad_f32_blocks(P);  // P = 0: one block writes zeros
    wgrad_f32_kernel<<<nblk, 64 * kWgWaves, 0, st>>>(dz, act, P, rg, part);
    slice_sum(part, nblk, kWgSlice, 65536, 256, dW, db, st);
}

void launch_slice_sum(const float* part, int nb, int64_t cols, float* out, hipStream_t st) {
    slice_sum(part, nb, cols, cols, 0, out, nullptr, st);
}

// Whole rounds of blocks over the compute units, the strips of 16 dealt evenly over them (at most 8 to a block): us at
// 8 queries of 2k / 10k / 20k / 50k Gaussians 21 / 31 / 42 / 55, with 8 strips to every block 49 / 51 / 49 / 57. 10k
// Gaussians are 625 strips, two or three to each of 256 blocks instead of eight to 79 of them.
int layer1_grad_blocks(int N) {
    const int strips = (N + 15) / 16, cus = n_compute_units();
    const int rounds = (strips + kL1Waves * cus - 1) / (kL1Waves * cus);
    return std::min(strips, rounds * cus);
}

void launch_layer1_grad(const void* dz1, const void* wf, const void* act, int B, int N, const RowGroups& rg, float* S,
                        float* Rpart, hipStream_t st) {
    if (N > 0 && B > 0)
        layer1_grad_kernel<<<layer1_grad_blocks(N), 64 * kL1Waves, 0, st>>>(
            (const __bf16*)dz1, (const uint4*)wf, (const __bf16*)act, B, N, rg.bits, S, Rpart);
}

int layer1_sums_blocks(int N) { return (N + kSumRows - 1) / kSumRows; }

void launch_layer1_sums(const float* z, const void* act, const uint32_t* bits, int B, int N, float* S, float* Rpart,
                        hipStream_t st) {
    if (N <= 0 || B <= 0) return;
    if (act)
        layer1_sums_kernel<true><<<layer1_sums_blocks(N), 256, 0, st>>>(z, (const __bf16*)act, bits, B, N, S, Rpart);
    else
        layer1_sums_kernel<false><<<layer1_sums_blocks(N), 256, 0, st>>>(z, nullptr, bits, B, N, S, Rpart);
}

void launch_to_bf16(const float* x, int64_t n, void* y, hipStream_t st) {
    if (n > 0) to_bf16_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(x, n, (__bf16*)y);
}

int mean_grad_blocks(int64_t N) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(512, (N + kMgRows - 1) / kMgRows));
}
size_t mean_grad_floats(int64_t N) { return (size_t)mean_grad_blocks(N) * kMgSlice; }

void launch_mean_grad(const float* S, const DevScene& d, float* part, float* dW, float* db, float* dmu,
                      hipStream_t st) {
    const int nb = mean_grad_blocks(d.n);  // no Gaussians: one block writes zeros
    mean_grad_kernel<<<nb, 256, 0, st>>>(S, d.w[0], d.in_dim, d.mx, d.my, d.n, d.W, d.H, dmu, part);
    slice_sum(part, nb, kMgSlice, 256 * kMeanFeat, 256, dW, db, st, kMeanFeat, d.in_dim);
}

}  // namespace swf
