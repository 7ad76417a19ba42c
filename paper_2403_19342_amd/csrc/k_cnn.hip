// Learned warm start for the level-2 eigenproblems (an extension of the
// method, not in the paper): a 3-layer 3D CNN maps the standardised
// log-permeability patch of each 8^3 element (with a one-cell halo) to k
// cell vectors that start the element's eigensolve.
//
//   a1 = relu(conv([patch, c_0..c_{k-1}], W1) + b1)   1+k -> 32 channels, 10^3 -> 8^3
//   a2 = relu(conv(a1, W2) + b2)                      32 -> 32 channels, zero padding 1
//   X  = c + conv(a2, W3) + b3                        32 -> k channels, zero padding 1
//
// c_j are the k lowest cosine modes of the homogeneous element (the start
// block of the cold eigensolve), cos(pi p (x+1/2)/8) cos(pi q (y+1/2)/8)
// cos(pi r (z+1/2)/8), evaluated on the patch grid (cells -1..8) as input
// channels and on the element (cells 0..7) as the base the network corrects.
// k is even (2, 4, 6 or 8).
//
// conv is the 3x3x3 cross-correlation y[o][p] = sum_c sum_t W[o][c][t]
// x[c][p + t] with t = (dz, dy, dx) in {0,1,2}^3.  Weights are bfloat16
// values, every product is accumulated in float32; activations are float32.
//
// Parameter vector (flat, this order): W1[32][1+k][27], b1[32],
// W2[32][32][27], b2[32], W3[k][32][27], b3[k].
//
// Training loss of one element (S: weight diagonal tr K~ of the element's
// cells normalised to mean 1; Phi: the first k eigenvectors, scaled so that
// Phi^T S Phi = I): loss = || Phi - X^T C* ||_S^2 with
// C* = (X S X^T)^-1 X S Phi, the S-distance of Phi from span(X).  Its
// gradient is dloss/dX = -2 C* (S R)^T with R = Phi - X^T C* (C* minimises
// the inner problem).  The batch loss is the mean over elements.
#include "common.hpp"

namespace specmg {

constexpr int kCnnC = 32;         // hidden channels
constexpr int kCnnIn = 1000;      // 10^3 input patch
constexpr int kCnnTile = 1000;    // LDS tile per input channel (10^3, zero halo for padded layers)

__device__ __forceinline__ float bf_lo(uint32_t u) { return __builtin_bit_cast(float, u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __builtin_bit_cast(float, u & 0xFFFF0000u); }

// float -> bfloat16, round to nearest even (NaN kept quiet)
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

// cosine mode j (j < 8, by increasing p^2+q^2+r^2, ties x before y before z)
// at integer cell coordinates (x, y, z) of an 8^3 block (-1..8 on the patch
// grid), cos(pi p (x+1/2)/8) cos(pi q (y+1/2)/8) cos(pi r (z+1/2)/8) with
// p, q, r in {0, 1}: a product of 1-D factors, read from c1[x + 1] =
// cos(pi (x+1/2)/8) (a factor with exponent 0 is 1).
// (p, q, r) of mode j as bit j of three masks: p for j in {1, 4, 5, 7},
// q for {2, 4, 6, 7}, r for {3, 5, 6, 7}
__device__ __forceinline__ void cnn_mode_pqr(int j, int& p, int& q, int& r) {
    p = (0xB2 >> j) & 1;
    q = (0xD4 >> j) & 1;
    r = (0xE8 >> j) & 1;
}

// the 10 factors c1[0..9] for x = -1..8; every thread of the block calls it
__device__ __forceinline__ void cnn_cos_table(double* c1) {
    if (threadIdx.x < 10) c1[threadIdx.x] = cos(3.14159265358979323846 / 8.0 * ((int)threadIdx.x - 1 + 0.5));
    __syncthreads();
}

__device__ __forceinline__ float cnn_mode(const double* c1, int j, int x, int y, int z) {
    int p, q, r;
    cnn_mode_pqr(j, p, q, r);
    const double fx = p ? c1[x + 1] : 1.0, fy = q ? c1[y + 1] : 1.0, fz = r ? c1[z + 1] : 1.0;
    return (float)(fx * fy * fz);
}

// ---------------------------------------------------------------------------
// patches: log kappa on the element and its halo (the nearest boundary cell
// repeated outside the domain), standardised by the patch's own mean and
// standard deviation (population, 1e-6 under the root).  Optionally also the
// element's weight diagonal tr K~ = s_scale * kappa (s_scale = 3 / h^2), cell
// order x fastest.
__global__ __launch_bounds__(256) void k_cnn_patches(FineGeom g, const double* __restrict__ perm, int e0,
                                                     double s_scale, float* __restrict__ out,
                                                     double* __restrict__ s_out) {
    __shared__ double sv[kCnnIn];
    __shared__ double sred[4];
    const int e = e0 + blockIdx.x;
    const int ex = e % g.mx, ey = (e / g.mx) % g.my, ez = e / (g.mx * g.my);
    double s1 = 0.0;
    for (int t = threadIdx.x; t < kCnnIn; t += blockDim.x) {
        const int x = t % 10, y = (t / 10) % 10, z = t / 100;
        int gx = ex * 8 + x - 1, gy = ey * 8 + y - 1, gz = ez * 8 + z - 1;
        gx = gx < 0 ? 0 : (gx >= g.nx ? g.nx - 1 : gx);
        gy = gy < 0 ? 0 : (gy >= g.ny ? g.ny - 1 : gy);
        gz = gz < 0 ? 0 : (gz >= g.nz ? g.nz - 1 : gz);
        const double v = log(perm[(size_t)gx + (size_t)g.nx * ((size_t)gy + (size_t)g.ny * gz)]);
        sv[t] = v;
        s1 += v;
    }
    const double mu = block_sum(s1, sred) / kCnnIn;
    double s2 = 0.0;
    for (int t = threadIdx.x; t < kCnnIn; t += blockDim.x) s2 += (sv[t] - mu) * (sv[t] - mu);
    const double inv = 1.0 / sqrt(block_sum(s2, sred) / kCnnIn + 1e-6);
    for (int t = threadIdx.x; t < kCnnIn; t += blockDim.x)
        out[(size_t)blockIdx.x * kCnnIn + t] = (float)((sv[t] - mu) * inv);
    if (s_out) {
        for (int c = threadIdx.x; c < 512; c += blockDim.x) {
            const int x = ex * 8 + (c & 7), y = ey * 8 + ((c >> 3) & 7), z = ez * 8 + (c >> 6);
            s_out[(size_t)blockIdx.x * 512 + c] =
                s_scale * perm[(size_t)x + (size_t)g.nx * ((size_t)y + (size_t)g.ny * z)];
        }
    }
}

// ---------------------------------------------------------------------------
// Staging of input channel c of element e into a 10^3 LDS tile.
//   IN = 1: 8^3 input [e][CIN][512], zero halo (padded layers)
//   IN = 2: the network input: channel 0 the patch [e][1000], channel
//           c >= 1 the cosine mode c-1 on the patch grid
template <int IN>
__device__ __forceinline__ float stage_value(const float* xe, int c, int r, const double* c1) {
    const int X = r % 10 - 1, Y = (r / 10) % 10 - 1, Z = r / 100 - 1;
    if (IN == 1) {
        const bool in = X >= 0 && X < 8 && Y >= 0 && Y < 8 && Z >= 0 && Z < 8;
        return in ? xe[(size_t)c * 512 + X + 8 * Y + 64 * Z] : 0.0f;
    }
    return c == 0 ? xe[r] : cnn_mode(c1, c - 1, X, Y, Z);
}

// The first layer of the widest network (1 + 8 input channels: one more than
// the K slices of k_conv1_mfma hold), one element per workgroup, one output
// position per thread, all 32 outputs in registers.  The input channels are
// staged in LDS as 10^3 tiles.  Wp[(c*27 + t)*16 + o/2] holds the bf16 pair of
// outputs (o, o+1), even o in the low half; the address is the same in every
// lane, so the pairs come through scalar loads.
template <int CIN>
__global__ __launch_bounds__(512) void k_conv1(const float* __restrict__ x, const uint32_t* __restrict__ Wp,
                                               const float* __restrict__ bias, float* __restrict__ y) {
    constexpr int COUT = 32;
    __shared__ float tile[CIN * kCnnTile];
    __shared__ double c1[10];
    cnn_cos_table(c1);
    const int e = blockIdx.x;
    const int p = threadIdx.x;
    const int base = (p >> 6) * 100 + ((p >> 3) & 7) * 10 + (p & 7);
    float acc[COUT];
#pragma unroll
    for (int o = 0; o < COUT; ++o) acc[o] = bias[o];
    const float* xe = x + (size_t)e * kCnnIn;
    for (int t = threadIdx.x; t < CIN * kCnnTile; t += blockDim.x)
        tile[t] = stage_value<2>(xe, t / kCnnTile, t % kCnnTile, c1);
    __syncthreads();
#pragma unroll 1
    for (int c = 0; c < CIN; ++c) {
        const uint32_t* wc = Wp + (size_t)c * 27 * (COUT / 2);
        const float* tc = tile + c * kCnnTile + base;
#pragma unroll
        for (int t = 0; t < 27; ++t) {
            const float v = tc[(t / 9) * 100 + ((t / 3) % 3) * 10 + (t % 3)];
#pragma unroll
            for (int o = 0; o < COUT / 2; ++o) {
                const uint32_t u = wc[t * (COUT / 2) + o];
                acc[2 * o] += bf_lo(u) * v;
                acc[2 * o + 1] += bf_hi(u) * v;
            }
        }
    }
#pragma unroll
    for (int o = 0; o < COUT; ++o) y[((size_t)e * COUT + o) * 512 + p] = fmaxf(acc[o], 0.0f);
}

// ---------------------------------------------------------------------------
// The convolutions of the layers with 32 input channels (a dense
// contraction of K = 27 taps x 32 channels per output), on the bf16 matrix
// cores: v_mfma_f32_16x16x32_bf16, D[16 positions][16 outputs] +=
// A[16 positions][32 channels] B[32 channels][16 outputs] per tap.  Lane l
// supplies A row l%16, channels 8(l/16)..+7, and B column l%16, the same
// channels; it receives D rows 4(l/16)..+3 of column l%16.
// Each activation is split into a bf16 high part and the bf16 rounding of
// the remainder, and both pass through the MFMA: with the weights exactly
// bf16 the products keep about 16 significant bits of the float32
// activation (relative error near 2^-17), and every sum is float32.
// One element per workgroup of 8 waves; the element's input is staged in
// LDS as [part][padded position (10^3)][channel], zero halo, and wave w
// owns position tiles 4w..4w+3 (positions 16 tile + row, x fastest).
// mf[t][o][c] (bf16, c fastest, o < COUTP) holds the weights.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kMfPos = 1000;   // padded positions of the staged element

template <int COUT, int COUTP, int ACT>
__global__ __launch_bounds__(512) void k_conv_mfma(const float* __restrict__ x, const uint16_t* __restrict__ mf,
                                                   const float* __restrict__ bias, float* __restrict__ y) {
    static_assert(COUTP % 16 == 0 && COUT <= COUTP, "output tiles of 16");
    constexpr int NT = COUTP / 16;
    __shared__ uint4 tile[2 * kMfPos * 4];   // [part][position][4 x 8 channels]
    __shared__ double c1[10];
    if (ACT == 3) cnn_cos_table(c1);
    const int e = blockIdx.x;
    for (int i = threadIdx.x; i < 2 * kMfPos * 4; i += blockDim.x) tile[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    {
        const int p = threadIdx.x;   // one interior position per thread
        const int P = ((p >> 6) + 1) * 100 + (((p >> 3) & 7) + 1) * 10 + (p & 7) + 1;
        const float* xe = x + (size_t)e * 32 * 512 + p;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint32_t hw[4], lw[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const float v0 = xe[(size_t)(8 * g + 2 * h) * 512], v1 = xe[(size_t)(8 * g + 2 * h + 1) * 512];
                const uint16_t h0 = f2bf(v0), h1 = f2bf(v1);
                const uint16_t l0 = f2bf(v0 - bf2f(h0)), l1 = f2bf(v1 - bf2f(h1));
                hw[h] = (uint32_t)h0 | ((uint32_t)h1 << 16);
                lw[h] = (uint32_t)l0 | ((uint32_t)l1 << 16);
            }
            tile[P * 4 + g] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
            tile[(kMfPos + P) * 4 + g] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
        }
    }
    __syncthreads();
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int r = l & 15, g = l >> 4;
    int base[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int p = 16 * (4 * w + j) + r;
        base[j] = (p >> 6) * 100 + ((p >> 3) & 7) * 10 + (p & 7);
    }
    f32x4_t acc[4][NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int o = 16 * n + r;
        const float b0 = (bias && o < COUT) ? bias[o] : 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j][n] = f32x4_t{b0, b0, b0, b0};
    }
#pragma unroll 1
    for (int t = 0; t < 27; ++t) {
        const int off = (t / 9) * 100 + ((t / 3) % 3) * 10 + (t % 3);
        bf16x8_t bw[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n)
            bw[n] = __builtin_bit_cast(bf16x8_t,
                                       *(const uint4*)(mf + ((size_t)(t * COUTP + 16 * n + r) * 32 + 8 * g)));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int P = base[j] + off;
            const bf16x8_t ah = __builtin_bit_cast(bf16x8_t, tile[P * 4 + g]);
            const bf16x8_t al = __builtin_bit_cast(bf16x8_t, tile[(kMfPos + P) * 4 + g]);
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bw[n], acc[j][n], 0, 0, 0);
                acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bw[n], acc[j][n], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int o = 16 * n + r;
        if (o >= COUT) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p0 = 16 * (4 * w + j) + 4 * g;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = acc[j][n][i];
                if (ACT == 1) v[i] = fmaxf(v[i], 0.0f);
                if (ACT == 3) {
                    const int p = p0 + i;
                    v[i] += cnn_mode(c1, o, p & 7, (p >> 3) & 7, p >> 6);
                }
            }
            *(float4*)(y + ((size_t)e * COUT + o) * 512 + p0) = make_float4(v[0], v[1], v[2], v[3]);
        }
    }
}

// The first layer (C1 = 1 + k <= 8 input channels: the patch and the mode
// channels, valid 3x3x3 over the 10^3 patch grid) on the same matrix-core
// tile: K = 32 is 4 taps x 8 channels (channels >= C1 and the 28th tap are
// zero), so the 27 taps take 7 K-steps.  Lane l supplies tap 4 step + l/16.
// The patch is staged as [part][position (10^3)][8 channels] bf16.
// mf1[step][o][tap in step][8 channels] (bf16) holds the weights.
constexpr int kMf1Steps = 7;

template <int C1>
__global__ __launch_bounds__(512) void k_conv1_mfma(const float* __restrict__ x, const uint16_t* __restrict__ mf,
                                                    const float* __restrict__ bias, float* __restrict__ y) {
    static_assert(C1 <= 8, "at most 8 input channels");
    __shared__ uint4 tile[2 * kMfPos];   // [part][position]: 8 channels
    __shared__ double c1[10];
    cnn_cos_table(c1);
    const int e = blockIdx.x;
    const float* xe = x + (size_t)e * kCnnIn;
    for (int P = threadIdx.x; P < kMfPos; P += blockDim.x) {
        const int X = P % 10 - 1, Y = (P / 10) % 10 - 1, Z = P / 100 - 1;
        uint32_t hw[4], lw[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            float v[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int c = 2 * h + u;
                v[u] = c == 0 ? xe[P] : (c < C1 ? cnn_mode(c1, c - 1, X, Y, Z) : 0.0f);
            }
            const uint16_t h0 = f2bf(v[0]), h1 = f2bf(v[1]);
            const uint16_t l0 = f2bf(v[0] - bf2f(h0)), l1 = f2bf(v[1] - bf2f(h1));
            hw[h] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            lw[h] = (uint32_t)l0 | ((uint32_t)l1 << 16);
        }
        tile[P] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
        tile[kMfPos + P] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
    }
    __syncthreads();
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int r = l & 15, g = l >> 4;
    int base[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int p = 16 * (4 * w + j) + r;
        base[j] = (p >> 6) * 100 + ((p >> 3) & 7) * 10 + (p & 7);
    }
    f32x4_t acc[4][2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const float b0 = bias[16 * n + r];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j][n] = f32x4_t{b0, b0, b0, b0};
    }
#pragma unroll 1
    for (int st = 0; st < kMf1Steps; ++st) {
        const int t = 4 * st + g;   // this lane's tap (t = 27: zero weights)
        const int off = t < 27 ? (t / 9) * 100 + ((t / 3) % 3) * 10 + (t % 3) : 0;
        bf16x8_t bw[2];
#pragma unroll
        for (int n = 0; n < 2; ++n)
            bw[n] = __builtin_bit_cast(bf16x8_t,
                                       *(const uint4*)(mf + ((size_t)(st * 32 + 16 * n + r) * 4 + g) * 8));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int P = base[j] + off;
            const bf16x8_t ah = __builtin_bit_cast(bf16x8_t, tile[P]);
            const bf16x8_t al = __builtin_bit_cast(bf16x8_t, tile[kMfPos + P]);
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bw[n], acc[j][n], 0, 0, 0);
                acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bw[n], acc[j][n], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int o = 16 * n + r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p0 = 16 * (4 * w + j) + 4 * g;
            *(float4*)(y + ((size_t)e * 32 + o) * 512 + p0) =
                make_float4(fmaxf(acc[j][n][0], 0.0f), fmaxf(acc[j][n][1], 0.0f), fmaxf(acc[j][n][2], 0.0f),
                            fmaxf(acc[j][n][3], 0.0f));
        }
    }
}

// ---------------------------------------------------------------------------
// The data gradient of a layer with 32 input channels: the convolution of gy
// (CIN channels, zero halo) with the flipped weights, kept where the relu was
// open (mask > 0).  Gradients are not split into bf16 parts: products and sums
// are float32, on v_mfma_f32_16x16x4_f32, D[16 positions][16 outputs] += A[16
// positions][4 channels] B[4 channels][16 outputs] per tap; operand lanes as in
// k_conv_wgrad.  One element per workgroup, wave w owning position tiles
// 4w..4w+3; the element lies in LDS as [channel][padded position], the weights
// (packed in pairs of outputs, as k_conv1 reads them) come from the L2, three
// taps ahead of their use.
// As scalar products, all outputs of a position in a thread, 512 elements took 319
// us (32 channels, 45 TFLOP/s) and 71 (6); now 155 and 41.
constexpr int kBackPitch = 1012;   // 1000 positions; four channels' rows of 16 spread over the banks
template <int CIN>
__global__ __launch_bounds__(512) void k_conv_back(const float* __restrict__ gy, const uint32_t* __restrict__ Wp,
                                                   const float* __restrict__ mask, float* __restrict__ y) {
    constexpr int S = (CIN + 3) / 4;   // steps of four channels
    __shared__ __align__(16) float tile[4 * S * kBackPitch];
    const int e = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6, li = lane & 15, lk = lane >> 4;
    constexpr int GV = (CIN * 128 + 511) / 512;
    float4 gr[GV];
#pragma unroll
    for (int u = 0; u < GV; ++u) {
        const int i = t + 512 * u;
        gr[u] = i < CIN * 128 ? *(const float4*)(gy + (size_t)e * CIN * 512 + 4 * i) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    // weights of the taps (dz, dy, 0..2): channel 4 s + lk, outputs 16 n + li
    uint32_t wt[3][S][2];
    auto weights = [&](int zy) {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    const int c = 4 * s + lk;
                    wt[dx][s][n] = c < CIN ? Wp[(c * 27 + 3 * zy + dx) * 16 + 8 * n + (li >> 1)] : 0u;
                }
    };
    weights(0);
    for (int i = t; i < S * kBackPitch; i += 512) ((float4*)tile)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GV; ++u) {
        const int i = t + 512 * u, c = i >> 7, q = (i & 127) * 4;   // four cells along x
        if (i < CIN * 128) {
            float* d = tile + c * kBackPitch + ((q >> 6) + 1) * 100 + (((q >> 3) & 7) + 1) * 10 + (q & 7) + 1;
            d[0] = gr[u].x;
            d[1] = gr[u].y;
            d[2] = gr[u].z;
            d[3] = gr[u].w;
        }
    }
    __syncthreads();
    f32x4_t acc[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[j][n] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // tile 4 w + j: z = w, y = 2 j and 2 j + 1
    const float* base = tile + lk * kBackPitch + w * 100 + (li >> 3) * 10 + (li & 7);
#pragma unroll 1
    for (int zy = 0; zy < 9; ++zy) {
        float b[3][S][2];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int n = 0; n < 2; ++n) b[dx][s][n] = li & 1 ? bf_hi(wt[dx][s][n]) : bf_lo(wt[dx][s][n]);
        if (zy < 8) weights(zy + 1);
        const float* at = base + (zy / 3) * 100 + (zy % 3) * 10;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float a = at[4 * s * kBackPitch + 20 * j + dx];
#pragma unroll
                    for (int n = 0; n < 2; ++n)
                        acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[dx][s][n], acc[j][n], 0, 0, 0);
                }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const size_t i = ((size_t)e * 32 + 16 * n + li) * 512 + 16 * (4 * w + j) + 4 * lk;
            const float4 m = *(const float4*)(mask + i);
            *(float4*)(y + i) = make_float4(m.x > 0.0f ? acc[j][n][0] : 0.0f, m.y > 0.0f ? acc[j][n][1] : 0.0f,
                                            m.z > 0.0f ? acc[j][n][2] : 0.0f, m.w > 0.0f ? acc[j][n][3] : 0.0f);
        }
}

// ---------------------------------------------------------------------------
// Weight gradients: part[b][(t*COUT + o)*CIN + c] = sum over the elements of
// block b of sum_p gy[e][o][p] x[e][c][p + t] (padded coordinates), and
// part[b][COUT*CIN*27 + o] = sum_p gy[e][o][p].
//
// Per tap a product of COUT x positions by positions x CIN, on the float32
// matrix cores: v_mfma_f32_16x16x4_f32 takes four positions (of one x row) a
// step, A[output][position] and B[position][channel] straight from LDS, lane l
// supplying row or column l%16 and position l/16; it receives rows 4(l/16)..+3
// of column l%16.  Products and sums are float32, four products and one sum a
// step.  An element goes through LDS in two slabs of four z planes (outputs'
// gradients, and the input's six planes with their zero halo; the network's own
// input, mostly the modes that all elements share, stays whole); a
// wavefront owns dz, 16 channels and every other x row, and keeps its 9 taps x
// COUT x 16 sums in registers for all its elements.  LDS pitches are odd
// multiples of 4 words, so the 16 rows x 4 positions of an operand lie in 64
// different banks; the next slab is on its way to registers meanwhile.
// As scalar products, a (c, o) pair a thread with its 27 sums, the three layers
// of 512 elements took 545 (32 -> 32, 27 TFLOP/s), 387 (32 -> 6) and 128 us
// (7 -> 32); now 131, 72 and 89.
constexpr int kWgX = 604;   // LDS pitch of an input channel: 6 planes of 10 x 10
constexpr int kWgPatch = 1004;   // of a channel of the network's input, all 10 planes
constexpr int kWgG = 260;   // of an output's gradient: 4 planes of 8 x 8

template <int CIN, int COUT>
struct WgradShape {
    static constexpr int NC = CIN <= 16 ? 1 : 2, OT = COUT <= 16 ? 1 : 2;   // tiles of 16 channels, of 16 outputs
    static constexpr int WAVES = 6 * NC;                                    // dz, channel tile, row parity
    static_assert(CIN <= 32 && COUT <= 32, "two tiles of 16");
};

template <int CIN, int COUT, int IN>
__global__ __launch_bounds__((64 * WgradShape<CIN, COUT>::WAVES)) void k_conv_wgrad(
    const float* __restrict__ x, const float* __restrict__ gy, int count, int per_block, float* __restrict__ part,
    int pstride) {
    constexpr int NC = WgradShape<CIN, COUT>::NC, OT = WgradShape<CIN, COUT>::OT;
    constexpr int NT = 64 * WgradShape<CIN, COUT>::WAVES;
    constexpr int ESZ = IN == 1 ? CIN * 512 : kCnnIn;
    constexpr int XP = IN == 1 ? kWgX : kWgPatch;
    constexpr int XN = 16 * NC * XP, GN = 16 * OT * kWgG;
    constexpr int SUMS = 3 * NC * 9 * OT * 4 * 64;   // sums of the odd rows' wavefronts, at the end
    constexpr int LDS = XN + GN > SUMS ? XN + GN : SUMS;
    constexpr int XV = (CIN * 6 * 16 + NT - 1) / NT, GV = (COUT * 64 + NT - 1) / NT;
    __shared__ __align__(16) float lds[LDS];
    __shared__ float sbias[NT];
    __shared__ double c1[10];
    float* xt = lds;
    float* gt = lds + XN;
    cnn_cos_table(c1);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, li = lane & 15, lk = lane >> 4;
    const int dz = w % 3, ct = (w / 3) % NC, par = w / (3 * NC);
    for (int i = t; i < XN + GN; i += NT) lds[i] = 0.0f;   // halos, and the rows beyond CIN and COUT
    f32x4_t acc[9][OT];
#pragma unroll
    for (int i = 0; i < 9; ++i)
#pragma unroll
        for (int o = 0; o < OT; ++o) acc[i][o] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    float accb = 0.0f;
    constexpr int BSEG = NT / COUT;                 // threads that sum one output's gradient
    const int bo = t % COUT, bs = t / COUT;
    const int e_beg = blockIdx.x * per_block;
    const int e_end = min(count, e_beg + per_block);
    const int nslab = 2 * (e_end - e_beg);
    float4 xr[IN == 1 ? XV : 1], gr[GV];
    constexpr int PV = IN == 1 ? 1 : (kCnnIn + NT - 1) / NT;
    float pr[PV];
    if constexpr (IN == 2) {   // the mode channels, the same for every element
        __syncthreads();
        for (int i = t; i < (CIN - 1) * kCnnIn; i += NT)
            xt[(1 + i / kCnnIn) * XP + i % kCnnIn] = stage_value<2>(nullptr, 1 + i / kCnnIn, i % kCnnIn, c1);
    }
    // slab s: planes z0 - 1 .. z0 + 4 of the input's cells, z0 .. z0 + 3 of gy's
    auto load = [&](int s) {
        const size_t e = e_beg + (s >> 1);
        const int z0 = 4 * (s & 1);
        if constexpr (IN == 1) {
#pragma unroll
            for (int u = 0; u < XV; ++u) {
                const int i = t + NT * u, c = i / 96, q = i % 96, Z = z0 + q / 16 - 1;   // q: plane, then 4 cells
                xr[u] = i < CIN * 96 && Z >= 0 && Z < 8
                            ? *(const float4*)(x + e * ESZ + (size_t)c * 512 + Z * 64 + (q % 16) * 4)
                            : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        } else if (!(s & 1)) {
#pragma unroll
            for (int u = 0; u < PV; ++u) pr[u] = t + NT * u < kCnnIn ? x[e * ESZ + t + NT * u] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < GV; ++u) {
            const int i = t + NT * u;
            gr[u] = i < COUT * 64 ? *(const float4*)(gy + (e * COUT + i / 64) * 512 + z0 * 64 + (i % 64) * 4)
                                  : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    };
    auto stage = [&](int s) {
        if constexpr (IN == 1) {
#pragma unroll
            for (int u = 0; u < XV; ++u) {
                const int i = t + NT * u, c = i / 96, q = i % 96, cell = (q % 16) * 4;
                if (i < CIN * 96) {
                    float* d = xt + c * XP + (q / 16) * 100 + (cell / 8 + 1) * 10 + cell % 8 + 1;
                    d[0] = xr[u].x;
                    d[1] = xr[u].y;
                    d[2] = xr[u].z;
                    d[3] = xr[u].w;
                }
            }
        } else if (!(s & 1)) {
#pragma unroll
            for (int u = 0; u < PV; ++u)
                if (t + NT * u < kCnnIn) xt[t + NT * u] = pr[u];
        }
#pragma unroll
        for (int u = 0; u < GV; ++u) {
            const int i = t + NT * u;
            if (i < COUT * 64) *(float4*)(gt + i / 64 * kWgG + (i % 64) * 4) = gr[u];
        }
    };
    if (nslab > 0) load(0);
    __syncthreads();
#pragma unroll 1
    for (int s = 0; s < nslab; ++s) {
        stage(s);
        __syncthreads();
        if (s + 1 < nslab) load(s + 1);
        if (bs < BSEG)
            for (int i = bs; i < 256; i += BSEG) accb += gt[bo * kWgG + i];
#pragma unroll 1
        for (int r = par; r < 32; r += 2) {
            const int z = r >> 3, y = r & 7;
            float a[2][OT];
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int o = 0; o < OT; ++o) a[kk][o] = gt[(16 * o + li) * kWgG + r * 8 + 4 * kk + lk];
            const float* xc = xt + (16 * ct + li) * XP + (IN == 2 ? 400 * (s & 1) : 0) + (z + dz) * 100 + y * 10 + lk;
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk) {
                        const float bv = xc[dy * 10 + 4 * kk + dx];
#pragma unroll
                        for (int o = 0; o < OT; ++o)
                            acc[dy * 3 + dx][o] =
                                __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk][o], bv, acc[dy * 3 + dx][o], 0, 0, 0);
                    }
        }
        __syncthreads();
    }
    // odd rows' sums to the even rows' wavefronts, which write
    float* mine = lds + (size_t)(w % (3 * NC)) * (9 * OT * 4 * 64) + lane;
    if (par == 1)
#pragma unroll
        for (int i = 0; i < 9; ++i)
#pragma unroll
            for (int o = 0; o < OT; ++o)
#pragma unroll
                for (int r = 0; r < 4; ++r) mine[((i * OT + o) * 4 + r) * 64] = acc[i][o][r];
    sbias[t] = accb;
    __syncthreads();
    float* pb = part + (size_t)blockIdx.x * pstride;
    const int c = 16 * ct + li;
    if (par == 0 && c < CIN)
#pragma unroll
        for (int i = 0; i < 9; ++i)
#pragma unroll
            for (int o = 0; o < OT; ++o)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int oo = 16 * o + 4 * lk + r;
                    if (oo < COUT)
                        pb[((size_t)(dz * 9 + i) * COUT + oo) * CIN + c] =
                            acc[i][o][r] + mine[((i * OT + o) * 4 + r) * 64];
                }
    if (t < COUT) {
        float v = 0.0f;
        for (int k = 0; k < BSEG; ++k) v += sbias[k * COUT + t];
        pb[(size_t)COUT * CIN * 27 + t] = v;
    }
}

// grad = sum_b part[b] for the layer's k output rows (rows o >= k of a padded
// layer are dropped), part ordered as k_conv_wgrad writes it, grad as the
// parameter vector; fixed summation order.  A thread sums a quarter of the
// blocks, 16 loads in flight: 61 -> 5.3 us for 256 blocks of 27680 sums.
__global__ __launch_bounds__(256) void k_cnn_reduce(const float* __restrict__ part, int nblk, int pstride, int cin,
                                                    int cout, int k, float* __restrict__ grad) {
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane, nw = 27 * cout * cin;
    const int per = (nblk + 3) / 4, b0 = w * per, b1 = min(nblk, b0 + per);
    float s = 0.0f;
    if (i < nw + cout) {
#pragma unroll 16
        for (int b = b0; b < b1; ++b) s += part[(size_t)b * pstride + i];
    }
    red[w][lane] = s;
    __syncthreads();
    if (w != 0 || i >= nw + cout) return;
    s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if (i >= nw) {
        if (i - nw < k) grad[(size_t)k * cin * 27 + i - nw] = s;
        return;
    }
    const int c = i % cin, o = i / cin % cout, tap = i / (cin * cout);
    if (o < k) grad[((size_t)o * cin + c) * 27 + tap] = s;
}

// ---------------------------------------------------------------------------
// Subspace loss and its gradient w.r.t. X, one element per workgroup, one
// cell per thread; the small k x k systems in float64.
template <int KP>
__global__ __launch_bounds__(512) void k_cnn_loss(const float* __restrict__ X, const double* __restrict__ phi,
                                                  int ldphi, const double* __restrict__ s, int k, double inv_m,
                                                  double* __restrict__ loss_part, float* __restrict__ gX) {
    __shared__ double red[8][2 * KP * KP];
    __shared__ double sG[KP * KP], sB[KP * KP], sC[KP * KP];
    __shared__ double sred[8];
    const int e = blockIdx.x, c = threadIdx.x;
    const int lane = c & 63, w = c >> 6;
    const double sc = s[(size_t)e * 512 + c];
    const double mean_s = block_sum(sc, sred) / 512.0;
    const double sb = sc / mean_s, root = sqrt(mean_s);
    double xv[KP], pv[KP];
#pragma unroll
    for (int o = 0; o < KP; ++o) {
        xv[o] = o < k ? (double)X[((size_t)e * KP + o) * 512 + c] : 0.0;
        pv[o] = o < k ? phi[((size_t)e * ldphi + o) * 512 + c] * root : 0.0;
    }
#pragma unroll
    for (int o = 0; o < KP; ++o) {
#pragma unroll
        for (int q = 0; q < KP; ++q) {
            const double gv = wave_sum(sb * xv[o] * xv[q]);
            const double bv = wave_sum(sb * xv[o] * pv[q]);
            if (lane == 0) {
                red[w][o * KP + q] = gv;
                red[w][KP * KP + o * KP + q] = bv;
            }
        }
    }
    __syncthreads();
    if (c < 2 * KP * KP) {
        double t = 0.0;
        for (int ww = 0; ww < 8; ++ww) t += red[ww][c];
        if (c < KP * KP) sG[c] = t;
        else sB[c - KP * KP] = t;
    }
    __syncthreads();
    if (c == 0) {
        // C = G^-1 B by Cholesky of G (k x k), a tiny ridge keeps it definite
        double Lm[KP * KP];
        double tr = 0.0;
        for (int i = 0; i < k; ++i) tr += sG[i * KP + i];
        const double ridge = 1e-12 * tr / k + 1e-300;
        for (int i = 0; i < KP * KP; ++i) Lm[i] = 0.0;
        for (int j = 0; j < k; ++j) {
            double d = sG[j * KP + j] + ridge;
            for (int l = 0; l < j; ++l) d -= Lm[j * KP + l] * Lm[j * KP + l];
            d = sqrt(fmax(d, 1e-300));
            Lm[j * KP + j] = d;
            for (int i = j + 1; i < k; ++i) {
                double v = sG[i * KP + j];
                for (int l = 0; l < j; ++l) v -= Lm[i * KP + l] * Lm[j * KP + l];
                Lm[i * KP + j] = v / d;
            }
        }
        for (int col = 0; col < KP; ++col) {
            double yv[KP];
            for (int i = 0; i < k; ++i) {
                double v = sB[i * KP + col];
                for (int l = 0; l < i; ++l) v -= Lm[i * KP + l] * yv[l];
                yv[i] = v / Lm[i * KP + i];
            }
            for (int i = k - 1; i >= 0; --i) {
                double v = yv[i];
                for (int l = i + 1; l < k; ++l) v -= Lm[l * KP + i] * sC[l * KP + col];
                sC[i * KP + col] = v / Lm[i * KP + i];
            }
            for (int i = k; i < KP; ++i) sC[i * KP + col] = 0.0;
        }
    }
    __syncthreads();
    double r[KP];
    double l2 = 0.0;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
        double v = pv[j];
#pragma unroll
        for (int o = 0; o < KP; ++o) v -= xv[o] * sC[o * KP + j];
        r[j] = j < k ? v : 0.0;
        l2 += sb * r[j] * r[j];
    }
#pragma unroll
    for (int o = 0; o < KP; ++o) {
        double gsum = 0.0;
#pragma unroll
        for (int j = 0; j < KP; ++j) gsum += sC[o * KP + j] * r[j];
        gX[((size_t)e * KP + o) * 512 + c] = o < k ? (float)(-2.0 * inv_m * sb * gsum) : 0.0f;
    }
    const double loss = block_sum(l2, sred);
    if (c == 0) loss_part[e] = loss * inv_m;
}

// ---------------------------------------------------------------------------
// Parameter packing for the convolution kernels.  Values come from the bf16
// vector or, rounded to bf16, from the float32 master vector.
//   fwd1[c][t][16], fwd2[c][t][16], fwd3[c][t][KP/2]       (pairs of outputs)
//   bwd2[o][t][16], bwd3[o][t][16] with flipped taps       (pairs of inputs)
//   mf2[t][32][32], mf3[t][16][32]: bf16 [tap][output][input] for the
//   matrix-core kernel (outputs of layer 3 beyond k are zero), 16-byte aligned;
//   mf1[step][32][4][8]: layer 1 as K-steps of 4 taps x 8 channels (zero
//   beyond C1 channels and beyond tap 26)
struct CnnPacks {
    uint32_t* fwd1;
    uint32_t* fwd2;
    uint32_t* fwd3;
    uint32_t* bwd2;
    uint32_t* bwd3;
    float* b1;
    float* b2;
    float* b3;
    uint16_t* mf2;
    uint16_t* mf3;
    uint16_t* mf1;
};

__device__ __forceinline__ float cnn_param(const float* t32, const uint16_t* t16, size_t i) {
    return t16 ? bf2f(t16[i]) : bf2f(f2bf(t32[i]));
}

__global__ void k_cnn_pack(const float* __restrict__ t32, const uint16_t* __restrict__ t16, int k, int kp,
                           CnnPacks pk) {
    const int c1 = 1 + k;   // input channels of layer 1
    const size_t oW1 = 0, ob1 = (size_t)32 * c1 * 27, oW2 = ob1 + 32, ob2 = oW2 + 32 * 32 * 27, oW3 = ob2 + 32,
                 ob3 = oW3 + (size_t)k * 32 * 27;
    auto W1 = [&](int o, int c, int t) { return cnn_param(t32, t16, oW1 + ((size_t)o * c1 + c) * 27 + t); };
    auto W2 = [&](int o, int c, int t) { return cnn_param(t32, t16, oW2 + ((size_t)o * 32 + c) * 27 + t); };
    auto W3 = [&](int o, int c, int t) {
        return o < k ? cnn_param(t32, t16, oW3 + ((size_t)o * 32 + c) * 27 + t) : 0.0f;
    };
    auto pack = [](float lo, float hi) {
        return (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
    };
    const int n1 = c1 * 27 * 16, n2 = 32 * 27 * 16, n3 = 32 * 27 * (kp / 2), nb2 = 32 * 27 * 16,
              nb3 = kp * 27 * 16;
    const int total = n1 + n2 + n3 + nb2 + nb3 + 32 + 32 + kp;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        int j = i;
        if (j < n1) {
            const int c = j / (27 * 16), t = (j / 16) % 27, op = j % 16;
            pk.fwd1[j] = pack(W1(2 * op, c, t), W1(2 * op + 1, c, t));
            continue;
        }
        j -= n1;
        if (j < n2) {
            const int c = j / (27 * 16), t = (j / 16) % 27, op = j % 16;
            pk.fwd2[j] = pack(W2(2 * op, c, t), W2(2 * op + 1, c, t));
            continue;
        }
        j -= n2;
        if (j < n3) {
            const int h = kp / 2;
            const int c = j / (27 * h), t = (j / h) % 27, op = j % h;
            pk.fwd3[j] = pack(W3(2 * op, c, t), W3(2 * op + 1, c, t));
            continue;
        }
        j -= n3;
        if (j < nb2) {
            // transposed layer 2: inputs o (32), outputs c (pairs), taps flipped
            const int o = j / (27 * 16), t = (j / 16) % 27, cp = j % 16;
            pk.bwd2[j] = pack(W2(o, 2 * cp, 26 - t), W2(o, 2 * cp + 1, 26 - t));
            continue;
        }
        j -= nb2;
        if (j < nb3) {
            const int o = j / (27 * 16), t = (j / 16) % 27, cp = j % 16;
            pk.bwd3[j] = pack(W3(o, 2 * cp, 26 - t), W3(o, 2 * cp + 1, 26 - t));
            continue;
        }
        j -= nb3;
        if (j < 32) {
            pk.b1[j] = cnn_param(t32, t16, ob1 + j);
            continue;
        }
        j -= 32;
        if (j < 32) {
            pk.b2[j] = cnn_param(t32, t16, ob2 + j);
            continue;
        }
        j -= 32;
        pk.b3[j] = j < k ? cnn_param(t32, t16, ob3 + j) : 0.0f;
    }
}

__global__ void k_cnn_pack_mf(const float* __restrict__ t32, const uint16_t* __restrict__ t16, int k,
                              CnnPacks pk) {
    const int c1 = 1 + k;
    const size_t oW2 = (size_t)32 * c1 * 27 + 32, oW3 = oW2 + 32 * 32 * 27 + 32;
    const int n2 = 27 * 32 * 32, n3 = 27 * 16 * 32, n1 = kMf1Steps * 32 * 4 * 8;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n2 + n3 + n1; i += gridDim.x * blockDim.x) {
        if (i >= n2 + n3) {
            const int j = i - n2 - n3, st = j / 1024, o = (j / 32) % 32, gg = (j / 8) % 4, c = j % 8;
            const int t = 4 * st + gg;
            pk.mf1[j] = (t < 27 && c < c1) ? f2bf(cnn_param(t32, t16, ((size_t)o * c1 + c) * 27 + t)) : (uint16_t)0;
        } else if (i < n2) {
            const int t = i / 1024, o = (i / 32) % 32, c = i % 32;
            pk.mf2[i] = f2bf(cnn_param(t32, t16, oW2 + ((size_t)o * 32 + c) * 27 + t));
        } else {
            const int j = i - n2, t = j / 512, o = (j / 32) % 16, c = j % 32;
            pk.mf3[j] = o < k ? f2bf(cnn_param(t32, t16, oW3 + ((size_t)o * 32 + c) * 27 + t)) : (uint16_t)0;
        }
    }
}

// Adam on the float32 master parameters; the bf16 copy used by inference
// is refreshed in the same pass.
__global__ void k_cnn_adam(float* __restrict__ theta, const float* __restrict__ grad, float* __restrict__ m1,
                           float* __restrict__ m2, int64_t n, float lr, float b1, float b2, float eps, float c1,
                           float c2, uint16_t* __restrict__ theta16) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float g = grad[i];
        const float a = b1 * m1[i] + (1.0f - b1) * g;
        const float b = b2 * m2[i] + (1.0f - b2) * g * g;
        m1[i] = a;
        m2[i] = b;
        const float v = theta[i] - lr * (a * c1) / (sqrtf(b * c2) + eps);
        theta[i] = v;
        if (theta16) theta16[i] = f2bf(v);
    }
}

// ---------------------------------------------------------------------------
// launchers

int64_t cnn_param_count(int k) {
    return (int64_t)32 * (1 + k) * 27 + 32 + 32 * 32 * 27 + 32 + (int64_t)k * 32 * 27 + k;
}

// 32-bit words of the packs before the matrix-core copies, rounded up to 16 bytes
static size_t cnn_pack_words_vec(int kp) {
    const size_t w = (size_t)(1 + kp) * 27 * 16 + 32 * 27 * 16 + 32 * 27 * (kp / 2) + 32 * 27 * 16 +
                     (size_t)kp * 27 * 16 + 32 + 32 + kp;
    return (w + 3) & ~(size_t)3;
}

size_t cnn_pack_words(int kp) {
    return cnn_pack_words_vec(kp) + (27 * 32 * 32 + 27 * 16 * 32 + kMf1Steps * 32 * 4 * 8) / 2;
}

CnnPacks cnn_pack_view(void* base, int kp) {
    CnnPacks p;
    uint32_t* u = (uint32_t*)base;
    p.fwd1 = u;
    p.fwd2 = p.fwd1 + (1 + kp) * 27 * 16;
    p.fwd3 = p.fwd2 + 32 * 27 * 16;
    p.bwd2 = p.fwd3 + 32 * 27 * (kp / 2);
    p.bwd3 = p.bwd2 + 32 * 27 * 16;
    p.b1 = (float*)(p.bwd3 + (size_t)kp * 27 * 16);
    p.b2 = p.b1 + 32;
    p.b3 = p.b2 + 32;
    p.mf2 = (uint16_t*)(u + cnn_pack_words_vec(kp));
    p.mf3 = p.mf2 + 27 * 32 * 32;
    p.mf1 = p.mf3 + 27 * 16 * 32;
    return p;
}

void launch_cnn_patches(const FineGeom& g, const double* perm, int e0, int count, double s_scale, float* out,
                        double* s_out, hipStream_t s) {
    hipLaunchKernelGGL(k_cnn_patches, dim3(count), dim3(256), 0, s, g, perm, e0, s_scale, out, s_out);
}

void launch_cnn_pack(const float* t32, const uint16_t* t16, int k, int kp, void* packs, hipStream_t s) {
    hipLaunchKernelGGL(k_cnn_pack, dim3(64), dim3(256), 0, s, t32, t16, k, kp, cnn_pack_view(packs, kp));
    hipLaunchKernelGGL(k_cnn_pack_mf, dim3(64), dim3(256), 0, s, t32, t16, k, cnn_pack_view(packs, kp));
}

#define SPECMG_KP_DISPATCH(KPV, ...)                                          \
    switch (KPV) {                                                            \
        case 2: { constexpr int KP = 2, C1 = 3; __VA_ARGS__; } break;         \
        case 4: { constexpr int KP = 4, C1 = 5; __VA_ARGS__; } break;         \
        case 6: { constexpr int KP = 6, C1 = 7; __VA_ARGS__; } break;         \
        default: { constexpr int KP = 8, C1 = 9; __VA_ARGS__; } break;        \
    }

// X = network(patches) for `count` elements; a1, a2 receive the hidden
// activations (kept for the backward pass)
void launch_cnn_forward(const void* packs, int kp, const float* patches, int count, float* a1, float* a2, float* X,
                        hipStream_t s) {
    const CnnPacks p = cnn_pack_view(const_cast<void*>(packs), kp);
    if (kp <= 6) {
        SPECMG_KP_DISPATCH(kp, hipLaunchKernelGGL((k_conv1_mfma<(C1 <= 8 ? C1 : 8)>), dim3(count), dim3(512), 0, s,
                                                  patches, p.mf1, p.b1, a1));
    } else {
        hipLaunchKernelGGL((k_conv1<9>), dim3(count), dim3(512), 0, s, patches, p.fwd1, p.b1, a1);
    }
    hipLaunchKernelGGL((k_conv_mfma<32, 32, 1>), dim3(count), dim3(512), 0, s, a1, p.mf2, p.b2, a2);
    SPECMG_KP_DISPATCH(kp, hipLaunchKernelGGL((k_conv_mfma<KP, 16, 3>), dim3(count), dim3(512), 0, s, a2, p.mf3,
                                              p.b3, X));
}

void launch_cnn_loss(const float* X, const double* phi, int ldphi, const double* sdiag, int k, int kp, int count,
                     double inv_m, double* loss_part, float* gX, hipStream_t s) {
    SPECMG_KP_DISPATCH(kp, hipLaunchKernelGGL((k_cnn_loss<KP>), dim3(count), dim3(512), 0, s, X, phi, ldphi,
                                              sdiag, k, inv_m, loss_part, gX));
}

// parameter gradient (flat, float32) from dL/dX; g2, g1: scratch of the
// activation size; part: scratch of nblk * (32*32*27 + 32) floats
void launch_cnn_backward(const void* packs, int k, int kp, const float* patches, const float* a1, const float* a2,
                         const float* gX, int count, float* g2, float* g1, float* part, int nblk, float* grad,
                         hipStream_t s) {
    const CnnPacks p = cnn_pack_view(const_cast<void*>(packs), kp);
    const int per = (count + nblk - 1) / nblk;
    const int nb = (count + per - 1) / per;
    const int64_t oW2 = (int64_t)32 * (1 + k) * 27 + 32, oW3 = oW2 + 32 * 32 * 27 + 32;
    auto reduce = [&](int cin, int cout, int rows, float* out) {
        hipLaunchKernelGGL(k_cnn_reduce, dim3((27 * cin * cout + cout + 63) / 64), dim3(256), 0, s, part, nb,
                           27 * cin * cout + cout, cin, cout, rows, out);
    };
    // layer 3: weight gradient, then data gradient through the relu of a2
    SPECMG_KP_DISPATCH(kp, hipLaunchKernelGGL((k_conv_wgrad<32, KP, 1>), dim3(nb), dim3(64 * WgradShape<32, KP>::WAVES), 0,
                                              s, a2, gX, count, per, part, 27 * 32 * KP + KP));
    reduce(32, kp, k, grad + oW3);
    SPECMG_KP_DISPATCH(kp, hipLaunchKernelGGL((k_conv_back<KP>), dim3(count), dim3(512), 0, s, gX, p.bwd3, a2, g2));
    // layer 2
    hipLaunchKernelGGL((k_conv_wgrad<32, 32, 1>), dim3(nb), dim3(64 * WgradShape<32, 32>::WAVES), 0, s, a1, g2, count, per,
                       part, 27 * 32 * 32 + 32);
    reduce(32, 32, 32, grad + oW2);
    hipLaunchKernelGGL((k_conv_back<32>), dim3(count), dim3(512), 0, s, g2, p.bwd2, a1, g1);
    // layer 1 (the network input needs no gradient)
    SPECMG_KP_DISPATCH(kp, hipLaunchKernelGGL((k_conv_wgrad<C1, 32, 2>), dim3(nb), dim3(64 * WgradShape<C1, 32>::WAVES), 0,
                                              s, patches, g1, count, per, part, 27 * 32 * C1 + 32));
    reduce(1 + k, 32, 32, grad);
}

void launch_cnn_adam(float* theta, const float* grad, float* m1, float* m2, int64_t n, float lr, float b1, float b2,
                     float eps, float c1, float c2, uint16_t* theta16, hipStream_t s) {
    hipLaunchKernelGGL(k_cnn_adam, dim3(64), dim3(256), 0, s, theta, grad, m1, m2, n, lr, b1, b2, eps, c1, c2,
                       theta16);
}

}  // namespace specmg
