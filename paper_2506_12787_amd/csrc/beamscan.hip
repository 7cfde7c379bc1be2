// Beam-scan spatial spectrum from multipath lists (paper Sec. 3.1): the
// receiver's sqrt(K) x sqrt(K) planar array, the per-element narrowband channel
// h_mn summed over the paths (received-signal equation, with the phase shift of
// the phase-shift equation), and the beam-scan spectrum A(theta, phi) =
// |(1/K) sum_mn w_mn(theta, phi) exp(j angle h_mn)| with the steering weights
// w_mn = exp(-j dalpha_mn(theta, phi)).
//
// Element (m, n) sits at r cos(theta - beta) = D ((n-1) cos theta + (m-1) sin theta), so every phase separates:
// exp(j dalpha_mn) = zu^(n-1) zv^(m-1) with zu, zv of the two axes alone. Two kernels per batch of queries:
//  1. channel_kernel: one wave per query. Lane l forms zu, zv of path l and their powers in FP64 (two complex
//     exponentials per path) into LDS; lane k < K then sums h_k over the paths by complex products and stores the
//     unit phasor c_k = h_k / |h_k| (0 where h_k = 0, whose angle is undefined) as FP32. FP64 keeps the phase of a
//     nearly cancelling h_k accurate. With the exponential of every (element, path) taken on its own, 25 of them one
//     after the other per lane, a batch of 256 queries took 21 us.
//  2. spectrum_kernel: the K-term sum of every (query, pixel) is a matrix product, on v_mfma_f32_16x16x4_f32 (FP32
//     products and sums): the rows are (query, re / im), the columns pixels, the contraction the 2 K real and
//     imaginary parts of the steering. A wave forms the steering of 32 pixels in registers in B-operand order (four
//     sincospi per pixel, dealt over the lanes that share it, then powers) and takes it through the query rows of its
//     block, whose phasors are in LDS in A-operand order; a lane's four results are (re, im) of two queries at one
//     pixel. Horner's rule on the vector ALUs (80 FMA per pixel and query at 4 x 4 elements) took 29 us for 256
//     queries of 90 x 360, bound by the FMA rate; the product needs 6.8 us of the matrix cores and 6.9 us of HBM
//     writes; it takes 19.
#include <math.h>

#include <type_traits>

#include "runtime.h"

namespace swf {

namespace {

constexpr int kMaxSide = 8;  // K <= 64: one lane per element in the channel kernel
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(64) void channel_kernel(const float* __restrict__ paths,
                                                     const int32_t* __restrict__ counts, int max_paths, int side,
                                                     double d_over_lambda, float2* __restrict__ phasor) {
    constexpr int kPaths = 32;  // paths per pass
    __shared__ double2 pu[kPaths][kMaxSide], pv[kPaths][kMaxSide];  // zu^n, zv^m
    __shared__ double s_rho[kPaths];
    const int q = blockIdx.x;
    const int k = threadIdx.x;
    const int K = side * side;
    const int L = min(max(counts[q], 0), max_paths);  // a count outside [0, max_paths] is clamped
    const int m = k / side, n = k - m * side;  // element (m + 1, n + 1), m-major
    const float* p = paths + (size_t)q * max_paths * 3;
    double re = 0.0, im = 0.0;
    for (int l0 = 0; l0 < L; l0 += kPaths) {
        const int nl = min(kPaths, L - l0);
        // lanes 2 l and 2 l + 1: the powers along n and along m of path l
        const int l = l0 + (k >> 1);
        if ((k >> 1) < nl) {
            const double rho = (double)p[3 * l], th = (double)p[3 * l + 1], ph = (double)p[3 * l + 2];
            // dalpha / pi = 2 (D / lambda) * (-r cos(theta - beta) cos phi) / D
            double s, c;
            sincospi(-2.0 * d_over_lambda * cos(ph) * (k & 1 ? sin(th) : cos(th)), &s, &c);
            double2* row = k & 1 ? pv[k >> 1] : pu[k >> 1];
            if (k & 1) s_rho[k >> 1] = rho;
            double2 z = make_double2(1.0 + 0.0 * c, 0.0);  // a non-finite angle reaches every element
            for (int i = 0; i < side; ++i) {
                row[i] = z;
                z = make_double2(z.x * c - z.y * s, z.x * s + z.y * c);
            }
        }
        __syncthreads();
        if (k < K)
            for (int i = 0; i < nl; ++i) {
                const double2 a = pu[i][n], b = pv[i][m];
                re += s_rho[i] * (a.x * b.x - a.y * b.y);
                im += s_rho[i] * (a.x * b.y + a.y * b.x);
            }
        __syncthreads();
    }
    if (k >= K) return;
    const double mag = hypot(re, im);
    float2 out = make_float2(0.f, 0.f);
    if (mag > 0.0) out = make_float2((float)(re / mag), (float)(im / mag));
    phasor[(size_t)q * K + k] = out;
}

// |re + j im| of a sum of unit phasors (0 exactly for 0): the hardware's reciprocal root and one correction, half the
// instructions of sqrtf, which also covers denormals
__device__ __forceinline__ float modulus(float re, float im) {
    const float x = fmaf(re, re, im * im);
    const float y = __builtin_amdgcn_rsqf(fmaxf(x, 1e-37f)), s = x * y;
    return fmaf(fmaf(-s, s, x), 0.5f * y, s);
}

constexpr int kWaves = 4;
constexpr int kPix = 2;  // 16-pixel tiles per wave

// Contraction index 4 c + g (chunk c, lane group g = lane / 16): element
// 2 c + g / 2, real part for even g, imaginary for odd. Row r of a query tile:
// query r / 2, the sum's real part for even r, imaginary for odd.
template <int SIDE>
__global__ __launch_bounds__(64 * kWaves) void spectrum_kernel(const float2* __restrict__ phasor, int B, int H, int W,
                                                               float two_d, float* __restrict__ out) {
    constexpr int K = SIDE * SIDE;
    constexpr int C = (K + 1) / 2;               // chunks
    constexpr int kTiles = SIDE <= 5 ? 8 : 4;    // query tiles (8 queries) per block
    __shared__ float sa[kTiles][C][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, col = lane & 15;
    const int q0 = blockIdx.y * kTiles * 8;
    const int tiles = min(kTiles, (B - q0 + 7) / 8);
    // phasor (q, e) is four operands: re = cr sr - ci si, im = ci sr + cr si
    for (int i = threadIdx.x; i < tiles * 8 * 2 * C; i += 64 * kWaves) {
        const int ql = i / (2 * C), e = i - ql * (2 * C);
        float2 p = make_float2(0.0f, 0.0f);
        if (q0 + ql < B && e < K) p = phasor[(size_t)(q0 + ql) * K + e];
        float* d = &sa[ql >> 3][e >> 1][32 * (e & 1) + 2 * (ql & 7)];
        d[0] = p.x;
        d[1] = p.y;
        d[16] = -p.y;
        d[17] = p.x;
    }
    const int HW = H * W;  // at most 2^24
    const int wpix = ((int)blockIdx.x * kWaves + wave) * (16 * kPix), pix0 = wpix + col;
    float b[kPix][C];
#pragma unroll
    for (int k = 0; k < kPix; ++k) {
        const uint32_t pix = (uint32_t)min(pix0 + 16 * k, HW - 1);
        const int y = (int)(pix / (uint32_t)W), x = (int)pix - y * W;
        // theta = 2 pi x / W (azimuth), phi = (pi / 2) y / H (elevation): even lane groups take theta and then zu,
        // odd ones phi and then zv
        const bool odd = g & 1;
        float s0, c0, s1, c1;
        sincospif(odd ? 0.5f * (float)y / (float)H : 2.0f * (float)x / (float)W, &s0, &c0);
        const float s2 = __shfl_xor(s0, 16), c2 = __shfl_xor(c0, 16);
        const float st = odd ? s2 : s0, ct = odd ? c2 : c0, cp = odd ? c0 : c2;
        // the phase (units of pi) as a rounded product and its remainder, which corrects the sine and cosine to first
        // order: the powers multiply the phase's error by up to SIDE - 1
        const float a = two_d * cp, t = odd ? st : ct, ph = a * t;
        const float lo = 3.14159265f * fmaf(fmaf(two_d, cp, -a), t, fmaf(a, t, -ph));
        float sp, cph;
        sincospif(ph, &sp, &cph);
        s1 = fmaf(lo, cph, sp);
        c1 = fmaf(-lo, sp, cph);
        const float s3 = __shfl_xor(s1, 16), c3 = __shfl_xor(c1, 16);
        const float ur = odd ? c3 : c1, ui = odd ? s3 : s1, vr = odd ? c1 : c3, vi = odd ? s1 : s3;
        if constexpr (K & 1) b[k][C - 1] = 0.0f;
        // powers by halves (zu^n = zu^(n/2) zu^(n - n/2)): three roundings deep at most
        float pr[SIDE], pi[SIDE], qr[SIDE], qi[SIDE];  // zu^n, zv^m
        pr[0] = qr[0] = 1.0f;
        pi[0] = qi[0] = 0.0f;
        if constexpr (SIDE > 1) {
            pr[1] = ur;
            pi[1] = ui;
            qr[1] = vr;
            qi[1] = vi;
        }
#pragma unroll
        for (int n = 2; n < SIDE; ++n) {
            const int i = n / 2, j = n - n / 2;
            pr[n] = pr[i] * pr[j] - pi[i] * pi[j];
            pi[n] = pr[i] * pi[j] + pi[i] * pr[j];
            qr[n] = qr[i] * qr[j] - qi[i] * qi[j];
            qi[n] = qr[i] * qi[j] + qi[i] * qr[j];
        }
#pragma unroll
        for (int e = 0; e < K; ++e) {
            const int m = e / SIDE, n = e % SIDE;
            const float er = m && n ? qr[m] * pr[n] - qi[m] * pi[n] : (m ? qr[m] : pr[n]);
            const float ei = m && n ? qr[m] * pi[n] + qi[m] * pr[n] : (m ? qi[m] : pi[n]);
            const float v = odd ? ei : er;
            if (e & 1)
                b[k][e / 2] = g >> 1 ? v : b[k][e / 2];
            else
                b[k][e / 2] = g >> 1 ? 0.0f : v;
        }
    }
    __syncthreads();
    const auto take = [&](auto whole) {  // whole tiles (the usual case) need no bounds per value
        float* o = out + (size_t)(q0 + 2 * g) * HW + pix0;
        for (int t = 0; t < tiles; ++t, o += (size_t)8 * HW) {
            // the sum in parts: shorter chains, and the partial sums' rounding stays below that of Horner's rule
            constexpr int kParts = C >= 12 ? 4 : (C > 1 ? 2 : 1);
            f32x4 part[kParts][kPix], acc[kPix];
#pragma unroll
            for (int c = 0; c < kParts * kPix; ++c) part[c / kPix][c % kPix] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float w = sa[t][c][lane];
#pragma unroll
                for (int k = 0; k < kPix; ++k) {
                    f32x4& s = part[c * kParts / C][k];
                    s = __builtin_amdgcn_mfma_f32_16x16x4f32(w, b[k][c], s, 0, 0, 0);
                }
            }
#pragma unroll
            for (int k = 0; k < kPix; ++k) {
                acc[k] = part[0][k];
                if constexpr (kParts == 2) acc[k] += part[1][k];
                if constexpr (kParts == 4) acc[k] = (part[0][k] + part[1][k]) + (part[2][k] + part[3][k]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float* oi = o + (size_t)i * HW;
#pragma unroll
                for (int k = 0; k < kPix; ++k) {
                    const float re = acc[k][2 * i], im = acc[k][2 * i + 1];
                    const float v = modulus(re, im) * (1.0f / (float)K);
                    if (whole || (q0 + 8 * t + 2 * g + i < B && pix0 + 16 * k < HW)) oi[16 * k] = v;
                }
            }
        }
    };
    if (wpix + 16 * kPix <= HW && q0 + 8 * tiles <= B)
        take(std::true_type{});
    else
        take(std::false_type{});
}

template <int SIDE>
void launch_spectrum(const float2* phasor, int B, int H, int W, float two_d, float* out, hipStream_t st) {
    const int64_t HW = (int64_t)H * W;
    constexpr int kQ = (SIDE <= 5 ? 8 : 4) * 8, kP = kWaves * 16 * kPix;
    dim3 grid((unsigned)((HW + kP - 1) / kP), (unsigned)((B + kQ - 1) / kQ));
    spectrum_kernel<SIDE><<<grid, 64 * kWaves, 0, st>>>(phasor, B, H, W, two_d, out);
}

}  // namespace

}  // namespace swf

using namespace swf;

extern "C" swf_status swf_beamscan(swf_ctx* h, const float* paths, const int32_t* counts, int32_t batch,
                                   int32_t max_paths, int32_t side, float spacing_over_lambda, int32_t height,
                                   int32_t width, float* out, void* stream) {
    Ctx* c = reinterpret_cast<Ctx*>(h);
    if (!c) return SWF_E_INVALID;
    std::lock_guard<std::recursive_mutex> lock(c->mu);
    hipSetDevice(c->device);
    if (batch < 1 || batch > 65535) return c->fail(SWF_E_INVALID, "batch must be in [1, 65535]");
    if (max_paths < 0) return c->fail(SWF_E_INVALID, "max_paths must be >= 0");
    if (side < 1 || side > kMaxSide) return c->fail(SWF_E_INVALID, "side must be in [1, 8]");
    if (!(spacing_over_lambda > 0.f) || !isfinite(spacing_over_lambda))
        return c->fail(SWF_E_INVALID, "spacing_over_lambda must be finite and > 0");
    if (height < 1 || height > 4096 || width < 1 || width > 4096)
        return c->fail(SWF_E_INVALID, "height and width must be in [1, 4096]");
    if (!counts || !out || (max_paths > 0 && !paths)) return c->fail(SWF_E_INVALID, "null pointer");
    hipStream_t st = (hipStream_t)stream;
    const int K = side * side;
    swf_status s = c->ws.beam.reserve(c, (size_t)batch * K * sizeof(float2), st);
    if (s) return s;
    float2* ph = (float2*)c->ws.beam.ptr;
    channel_kernel<<<batch, 64, 0, st>>>(paths, counts, max_paths, side, (double)spacing_over_lambda, ph);
    const float two_d = 2.0f * spacing_over_lambda;
    switch (side) {
        case 1: launch_spectrum<1>(ph, batch, height, width, two_d, out, st); break;
        case 2: launch_spectrum<2>(ph, batch, height, width, two_d, out, st); break;
        case 3: launch_spectrum<3>(ph, batch, height, width, two_d, out, st); break;
        case 4: launch_spectrum<4>(ph, batch, height, width, two_d, out, st); break;
        case 5: launch_spectrum<5>(ph, batch, height, width, two_d, out, st); break;
        case 6: launch_spectrum<6>(ph, batch, height, width, two_d, out, st); break;
        case 7: launch_spectrum<7>(ph, batch, height, width, two_d, out, st); break;
        default: launch_spectrum<8>(ph, batch, height, width, two_d, out, st); break;
    }
    return c->hip(hipGetLastError(), "beam-scan launch");
}
