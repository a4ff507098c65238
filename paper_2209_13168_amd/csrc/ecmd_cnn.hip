// Learned-incumbent network of the divergence estimator (gfx950).
//
// A small convolutional regressor proposes a divergence for each window from
// its unwarped 64x64 event-count image; the proposal seeds the incumbent of
// the branch and bound, which still certifies the optimum.  Layers:
//   conv3x3/s2/p1 1->16, ReLU (32x32), conv3x3/s2/p1 16->32, ReLU (16x16),
//   conv3x3/s2/p1 32->64, ReLU (8x8), mean over positions, linear 64->1.
// Weights and layer inputs are rounded to bfloat16 (nearest even) where they
// enter a product; products and sums are fp32.  The backward pass treats the
// rounding as the identity.  One workgroup per image keeps every activation
// of that image in LDS; parameters are read from HBM/L2.
#include "ecmd_internal.hpp"

namespace ecmd {

namespace cnn {
constexpr int oW1 = 0, oB1 = oW1 + 16 * 1 * 9, oW2 = oB1 + 16, oB2 = oW2 + 32 * 16 * 9, oW3 = oB2 + 32,
              oB3 = oW3 + 64 * 32 * 9, oWfc = oB3 + 64, oBfc = oWfc + 64, kNParam = oBfc + 1;
static_assert(kNParam == 23361, "parameter count");
}  // namespace cnn

using namespace cnn;

__device__ __forceinline__ float bf(float v) {
    unsigned u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return __uint_as_float(u & 0xFFFF0000u);
}

__device__ __forceinline__ float bits_to_f(uint16_t b) { return __uint_as_float((unsigned)b << 16); }

// ------------------------------------------------------------ one image per workgroup
//
// One workgroup of 16 waves keeps every activation of its image in LDS.  A
// layer's planes carry a zero row above and a zero column to the left, so a
// tap needs no range test; read one past its end, a plane's row continues in
// the next row's zero column and the plane in the next plane's zero row (one
// more row of zeros after the last), which is the border that the transposed
// products of the backward pass need.
//
// The second and third convolution and the products of the backward pass run
// on v_mfma_f32_16x16x4_f32: fp32 products and sums, as the rounding rules
// above ask for (gradients are not rounded, so they take fp32).  It adds its
// four products one after another with one rounding each, so an output of the
// forward pass is the chain of fused multiply-adds over its weights' order,
// whichever kernel computes it (a tap on the zero border adds nothing).
//
// The floor is the matrix cores' fp32 rate: an image's forward pass is 2304
// MFMA of 32 cycles over a CU's four SIMDs (8 us at 2.4 GHz), its backward
// pass 4864 (16 us).  Measured 33 us forward (64 images) and 81 us forward and
// backward (256): bound by the products' operands, which come through LDS, by
// the parts in which the weights are staged (a barrier before and after each,
// nothing in flight across it) and by the layers following one another.
constexpr int kImgThreads = 1024;
constexpr int kImgWaves = kImgThreads / 64;
constexpr int kI = 65, kP1 = 33, kP2 = 17, kP3 = 9;       // row lengths of the planes
constexpr int kN1 = kP1 * kP1, kN2 = kP2 * kP2, kN3 = kP3 * kP3;
// row lengths of the staged weights (odd: no bank conflicts): conv2's, 16 output
// channels of conv3's, 8 input channels of conv3's
constexpr int kWs2 = 145, kWs3 = 289, kWs3f = 73;
// LDS (floats): image (bfloat16 bits), a1, a2, a3, staged weights, tap offsets, scratch
constexpr int tA1 = (kI * kI + 1) / 2, tA2 = tA1 + 16 * kN1, tA3 = tA2 + 32 * kN2 + kP2 + 1,
              tW = tA3 + 64 * kN3 + kP3 + 1, tTab = tW + 64 * kWs3f, tRed = tTab + 144 + 288,
              kLdsFloats = tRed + 65;
static_assert(64 * kWs3f >= 16 * kWs3 && 64 * kWs3f >= 32 * kWs2 && 64 * kWs3f >= kImgWaves * 256,
              "the staging area holds every part");

typedef float v4f __attribute__((ext_vector_type(4)));

// Lane l of a wave holds row l % 16 of A, column l % 16 of B, at k index
// l / 16, and column l % 16, rows 4 (l / 16) .. + 3 of the result.
__device__ __forceinline__ v4f mfma(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float wave_sum(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// The forward pass of image b up to a3 (unrounded), all planes in LDS at s;
// returns the prediction (wave 0 only), with the pooled values, rounded, in
// the scratch.
__device__ float forward(float* s, const float* __restrict__ P, const uint16_t* __restrict__ imgs, int b) {
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint16_t* const img = reinterpret_cast<uint16_t*>(s);
    float* const a1 = s + tA1;
    float* const a2 = s + tA2;
    float* const a3 = s + tA3;
    float* const ws = s + tW;
    int* const tab2 = reinterpret_cast<int*>(s + tTab);  // plane offset of weight k = 9 i + tap
    int* const tab3 = tab2 + 144;
    float* const red = s + tRed;
    // zero borders (everything but the scratch), tap offsets, then the image
    for (int k = tid; k < tW; k += kImgThreads) s[k] = 0.0f;
    for (int k = tid; k < 32 * 144; k += kImgThreads) ws[k / 144 * kWs2 + k % 144] = bf(P[oW2 + k]);
    if (tid < 144) tab2[tid] = tid / 9 * kN1 + tid % 9 / 3 * kP1 + tid % 3;
    if (tid < 288) tab3[tid] = tid / 9 * kN2 + tid % 9 / 3 * kP2 + tid % 3;
    __syncthreads();
    for (int k = tid; k < 4096; k += kImgThreads) img[(k / 64 + 1) * kI + k % 64 + 1] = imgs[(long long)b * 4096 + k];
    __syncthreads();
    {  // conv1: one position a thread, the 16 channels from nine image reads
        const int y = tid >> 5, x = tid & 31;
        float v[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) v[t] = bits_to_f(img[(2 * y + t / 3) * kI + 2 * x + t % 3]);
        for (int o = 0; o < 16; ++o) {
            float acc = 0.0f;
#pragma unroll
            for (int t = 0; t < 9; ++t) acc = fmaf(bf(P[oW1 + o * 9 + t]), v[t], acc);
            a1[o * kN1 + (y + 1) * kP1 + x + 1] = bf(fmaxf(acc + P[oB1 + o], 0.0f));
        }
    }
    __syncthreads();
    {  // conv2: 2 channel tiles x 16 rows, two rows a wave
        const int o = (wave & 1) * 16, y = wave >> 1;
        const float* const w = ws + (o + l16) * kWs2 + lg;
        const float* const in = a1 + 2 * y * kP1 + 2 * l16;
        v4f acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll 6
        for (int k = 0; k < 144; k += 4) {
            const float a = w[k];
            const float* const at = in + tab2[k + lg];
            acc[0] = mfma(a, at[0], acc[0]);
            acc[1] = mfma(a, at[16 * kP1], acc[1]);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = o + 4 * lg + r;
                a2[c * kN2 + (y + 8 * j + 1) * kP2 + l16 + 1] = bf(fmaxf(acc[j][r] + P[oB2 + c], 0.0f));
            }
    }
    {  // conv3: 4 channel tiles x 4 pairs of rows, the weights of 8 input channels at a time
        const int o = (wave & 3) * 16, p = (wave >> 2) * 16 + l16, y = p >> 3, x = p & 7;
        const float* const in = a2 + 2 * y * kP2 + 2 * x;
        const float* const w = ws + (o + l16) * kWs3f + lg;
        v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int k0 = 0; k0 < 288; k0 += 72) {
            __syncthreads();
            for (int k = tid; k < 64 * 72; k += kImgThreads)
                ws[k / 72 * kWs3f + k % 72] = bf(P[oW3 + k / 72 * 288 + k0 + k % 72]);
            __syncthreads();
#pragma unroll 6
            for (int k = 0; k < 72; k += 4) acc = mfma(w[k], in[tab3[k0 + k + lg]], acc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = o + 4 * lg + r;
            a3[c * kN3 + (y + 1) * kP3 + x + 1] = fmaxf(acc[r] + P[oB3 + c], 0.0f);
        }
    }
    __syncthreads();
    float d = 0.0f;
    if (wave == 0) {  // mean over positions, the last layer: sums in order
        float acc = 0.0f;
#pragma unroll 16
        for (int p = 0; p < 64; ++p) acc += a3[lane * kN3 + ((p >> 3) + 1) * kP3 + (p & 7) + 1];
        const float m = bf(acc * (1.0f / 64.0f));
        red[lane] = m;
        const float v = m * bf(P[oWfc + lane]);
#pragma unroll
        for (int c = 0; c < 64; ++c) d += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), c));
        d += P[oBfc];
    }
    return d;
}

// Per-image gradients of the MSE loss with `inv_n` = 1 / batch to
// pg[b][kNParam], the per-image loss to lossb[b], the prediction to out[b].
// Measured per training step of 256 images: 122 us against 1725 us with
// 256 threads an image and an fp32 fma per product and lane; gradients of 40
// images 108 us against 1980 us.
__global__ __launch_bounds__(kImgThreads) void k_cnn_train(const float* __restrict__ P,
                                                          const uint16_t* __restrict__ imgs, int B,
                                                          float* __restrict__ out, const float* __restrict__ labels,
                                                          float inv_n, float* __restrict__ pg,
                                                          float* __restrict__ lossb) {
    extern __shared__ float s[];
    const int b = blockIdx.x;
    if (b >= B) return;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint16_t* const img = reinterpret_cast<uint16_t*>(s);
    float* const a1 = s + tA1;
    float* const a2 = s + tA2;
    float* const a3 = s + tA3;
    float* const ws = s + tW;
    float* const red = s + tRed;
    float* const gp = pg + (long long)b * kNParam;

    float d = forward(s, P, imgs, b);
    if (tid == 0) red[64] = d;
    __syncthreads();
    d = red[64];
    const int p3 = ((lane >> 3) + 1) * kP3 + (lane & 7) + 1;  // position `lane` of the 8 x 8 planes
    const float err = d - labels[b];
    const float dd = 2.0f * err * inv_n;
    if (tid == 0) {
        out[b] = d;
        gp[oBfc] = dd;
        lossb[b] = err * err * inv_n;
    }
    if (tid < 64) gp[oWfc + tid] = dd * red[tid];
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // dz3 in place, and its sums
        const int c = wave * 4 + j;
        float* const z = a3 + c * kN3 + p3;
        const float v = *z > 0.0f ? dd * bf(P[oWfc + c]) * (1.0f / 64.0f) : 0.0f;
        *z = v;
        const float t = wave_sum(v);
        if (lane == 0) gp[oB3 + c] = t;
    }
    __syncthreads();
    {  // dW3[o][i][t] = sum_p dz3[o][p] a2[i][p, t]: 4 channel tiles x (9 taps x 2 input tiles)
        const int o = (wave & 3) * 16;
        float za[16];
        int pos[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int p = 4 * k + lg, y = p >> 3, x = p & 7;
            za[k] = a3[(o + l16) * kN3 + (y + 1) * kP3 + x + 1];
            pos[k] = 2 * y * kP2 + 2 * x;
        }
        for (int n = wave >> 2; n < 18; n += 4) {
            const int t = n >> 1, i = (n & 1) * 16 + l16;
            const float* const in = a2 + i * kN2 + t / 3 * kP2 + t % 3;
            v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 16; ++k) acc = mfma(za[k], in[pos[k]], acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) gp[oW3 + (o + 4 * lg + r) * 288 + i * 9 + t] = acc[r];
        }
    }
    {  // da2[i][iy, ix] = (a2 > 0) sum over output channels and the taps that reach (iy, ix).  An
       // even coordinate is reached by the middle tap alone, an odd one 2 q + 1 by
       // the first tap of q + 1 and the last of q.  Waves 0-7 take the positions
       // with both coordinates odd (4 taps) and both even (1), waves 8-15 the others (2 + 2).
        const int i0 = (wave & 1) * 16, q = ((wave >> 1) & 3) * 16 + l16, qy = q >> 3, qx = q & 7;
        const int half = wave >> 3;
        v4f acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
        for (int ob = 0; ob < 64; ob += 16) {  // 16 output channels' weights at a time
            __syncthreads();
            for (int k = tid; k < 16 * 288; k += kImgThreads) ws[k / 288 * kWs3 + k % 288] = bf(P[oW3 + ob * 288 + k]);
            __syncthreads();
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int oy = half == 0 ? 1 - c : c, ox = 1 - c;  // odd coordinates of this class
                for (int ty = 0; ty <= oy; ++ty)
                    for (int tx = 0; tx <= ox; ++tx) {
                        const int ky = oy ? 2 * ty : 1, kx = ox ? 2 * tx : 1;
                        const int sy = oy ? 1 - ty : 0, sx = ox ? 1 - tx : 0;
                        const float* const z = a3 + ob * kN3 + (qy + sy + 1) * kP3 + qx + sx + 1;
                        const float* const w = ws + (i0 + l16) * 9 + ky * 3 + kx;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            acc[c] = mfma(w[(4 * k + lg) * kWs3], z[(4 * k + lg) * kN3], acc[c]);
                    }
            }
        }
        // (every wave is past the weight gradient's reads of a2)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int oy = half == 0 ? 1 - c : c, ox = 1 - c;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float* const z = a2 + (i0 + 4 * lg + r) * kN2 + (2 * qy + oy + 1) * kP2 + 2 * qx + ox + 1;
                *z = *z > 0.0f ? acc[c][r] : 0.0f;
            }
        }
    }
    __syncthreads();
    // dW2[o][i][t] = sum_p dz2[o][p] a1[i][p, t]: 2 channel tiles x 9 taps, and dz2's sums
    for (int n = wave; n < 18; n += kImgWaves) {
        const int o = (n & 1) * 16, t = n >> 1;
        const float* const z = a2 + (o + l16) * kN2 + kP2 + 1;
        const float* const in = a1 + l16 * kN1 + t / 3 * kP1 + t % 3;
        v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
        for (int k = 0; k < 64; ++k) {
            const int y = k >> 2, x = (k & 3) * 4 + lg;
            acc = mfma(z[y * kP2 + x], in[2 * y * kP1 + 2 * x], acc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) gp[oW2 + (o + 4 * lg + r) * 144 + l16 * 9 + t] = acc[r];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int c = wave * 2 + j;
        float t = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) t += a2[c * kN2 + (k * 4 + lg + 1) * kP2 + l16 + 1];
        t = wave_sum(t);
        if (lane == 0) gp[oB2 + c] = t;
    }
    // the last reads of the staged weights lie before the barrier above
    for (int k = tid; k < 32 * 144; k += kImgThreads) ws[k / 144 * kWs2 + k % 144] = bf(P[oW2 + k]);
    __syncthreads();
    {  // da1, as da2: row q of every class, a wave each
        const int q = wave;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int oy = c >> 1, ox = c & 1;
            v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int ty = 0; ty <= oy; ++ty)
                for (int tx = 0; tx <= ox; ++tx) {
                    const int ky = oy ? 2 * ty : 1, kx = ox ? 2 * tx : 1;
                    const int sy = oy ? 1 - ty : 0, sx = ox ? 1 - tx : 0;
                    const float* const z = a2 + (q + sy + 1) * kP2 + l16 + sx + 1;
                    const float* const w = ws + l16 * 9 + ky * 3 + kx;
#pragma unroll
                    for (int k = 0; k < 8; ++k) acc = mfma(w[(4 * k + lg) * kWs2], z[(4 * k + lg) * kN2], acc);
                }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float* const z = a1 + (4 * lg + r) * kN1 + (2 * q + oy + 1) * kP1 + 2 * l16 + ox + 1;
                *z = *z > 0.0f ? acc[r] : 0.0f;
            }
        }
    }
    __syncthreads();
    {  // dW1[o][t] and (column 9) dz1's sums: each wave two rows, then the waves' sums
        const int t = l16 < 9 ? l16 : 0;
        v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int y = wave * 2 + (k >> 3), x = (k & 7) * 4 + lg;
            const float v = bits_to_f(img[(2 * y + t / 3) * kI + 2 * x + t % 3]);
            acc = mfma(a1[l16 * kN1 + (y + 1) * kP1 + x + 1], l16 < 9 ? v : 1.0f, acc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) ws[wave * 256 + (4 * lg + r) * 16 + l16] = acc[r];
    }
    __syncthreads();
    if (tid < 256) {
        const int o = tid >> 4, t = tid & 15;
        float v = 0.0f;
        for (int k = 0; k < kImgWaves; ++k) v += ws[k * 256 + tid];
        if (t < 9) gp[oW1 + o * 9 + t] = v;
        if (t == 9) gp[oB1 + o] = v;
    }
}

// Forward pass alone (the proposal of the learned incumbent).  Measured on 64
// images: 33 us, against 126 us with an fp32 fma per product and lane.
__global__ __launch_bounds__(kImgThreads) void k_cnn_fwd(const float* __restrict__ P,
                                                        const uint16_t* __restrict__ imgs, int B,
                                                        float* __restrict__ out) {
    extern __shared__ float s[];
    if ((int)blockIdx.x >= B) return;
    const float d = forward(s, P, imgs, blockIdx.x);
    if (threadIdx.x == 0) out[blockIdx.x] = d;
}

// grad[p] = sum_b pg[b][p], loss = sum_b lossb[b], in a fixed order: each wave
// of the workgroup sums every kRedWaves-th image of its 64 parameters, then
// the waves' sums are added.  HBM-bound: 8 images' reads in flight per wave.
constexpr int kRedWaves = 8;
__global__ __launch_bounds__(64 * kRedWaves) void k_cnn_reduce(const float* __restrict__ pg,
                                                               const float* __restrict__ lossb, int B,
                                                               float* __restrict__ grad, float* __restrict__ loss) {
    __shared__ float part[kRedWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    float acc = 0.0f;
    if (p < kNParam) {
#pragma unroll 8
        for (int b = wave; b < B; b += kRedWaves) acc += pg[(long long)b * kNParam + p];
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && p < kNParam) {
        float t = part[0][lane];
        for (int k = 1; k < kRedWaves; ++k) t += part[k][lane];
        grad[p] = t;
    }
    if (blockIdx.x == 0 && wave == 1) {
        float t = 0.0f;
        for (int b = lane; b < B; b += 64) t += lossb[b];
        t = wave_sum(t);
        if (lane == 0) *loss = t;
    }
}

__global__ void k_adam(float* __restrict__ P, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ grad, float lr, float c1, float c2) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kNParam) return;
    const float g = grad[p];
    const float mi = 0.9f * m[p] + 0.1f * g;
    const float vi = 0.999f * v[p] + 0.001f * g * g;
    m[p] = mi;
    v[p] = vi;
    P[p] -= lr * (mi * c1) / (sqrtf(vi * c2) + 1e-8f);
}

// Nearest grid index of each prediction as the seed divergence (NaN if not finite).
__global__ void k_seed_from_pred(const float* __restrict__ pred, int B, float d_lo, float d_hi,
                                 float* __restrict__ seeds) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const float d = pred[b];
    seeds[b] = isfinite(d) ? fminf(fmaxf(d, d_lo), d_hi) : __builtin_nanf("");
}

int cnn_nparam() { return kNParam; }

hipError_t cnn_set_lds() {
    const int bytes = kLdsFloats * sizeof(float);
    hipError_t e = hipFuncSetAttribute((const void*)k_cnn_train, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void*)k_cnn_fwd, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t launch_cnn(hipStream_t s, const float* P, const uint16_t* imgs, int B, float* out, int mode,
                      const float* labels, float* pg, float* lossb) {
    if (B <= 0) return hipSuccess;
    if (mode == 0)
        k_cnn_fwd<<<B, kImgThreads, kLdsFloats * sizeof(float), s>>>(P, imgs, B, out);
    else
        k_cnn_train<<<B, kImgThreads, kLdsFloats * sizeof(float), s>>>(P, imgs, B, out, labels, 1.0f / (float)B, pg,
                                                                        lossb);
    return hipGetLastError();
}

hipError_t launch_cnn_reduce(hipStream_t s, const float* pg, const float* lossb, int B, float* grad, float* loss) {
    k_cnn_reduce<<<(kNParam + 63) / 64, 64 * kRedWaves, 0, s>>>(pg, lossb, B, grad, loss);
    return hipGetLastError();
}

hipError_t launch_adam(hipStream_t s, float* P, float* m, float* v, const float* grad, float lr, int step) {
    const float c1 = 1.0f / (1.0f - powf(0.9f, (float)step));
    const float c2 = 1.0f / (1.0f - powf(0.999f, (float)step));
    k_adam<<<(kNParam + 255) / 256, 256, 0, s>>>(P, m, v, grad, lr, c1, c2);
    return hipGetLastError();
}

hipError_t launch_seed_from_pred(hipStream_t s, const float* pred, int B, float d_lo, float d_hi, float* seeds) {
    if (B <= 0) return hipSuccess;
    k_seed_from_pred<<<(B + 255) / 256, 256, 0, s>>>(pred, B, d_lo, d_hi, seeds);
    return hipGetLastError();
}

}  // namespace ecmd
