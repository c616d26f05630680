// Per-variable fix predictor on BF16 matrix cores (gfx950 MFMA):
//   h1 = relu(W1 f + b1), h2 = relu(W2 bf16(h1) + b2), logit = w3 . h2 + b3
// with 16 padded features, 64 hidden units per layer, FP32 accumulation.
//
// One wave evaluates 16 variables at a time in the transposed form
// H1^T (64 x 16) = W1 (64 x 16) F^T (16 x 16): with v_mfma_f32_16x16x16_bf16
// a lane holds A[row = lane % 16][k = 4 (lane / 16) + i], B[k = 4 (lane / 16)
// + i][col = lane % 16] and D[row = 4 (lane / 16) + i][col = lane % 16], so the
// D block of one layer is already the B operand of the next layer's K block
// and the layers chain in registers.  The 64-wide layer-2 contractions use
// gfx950's v_mfma_f32_16x16x32_bf16, two K = 32 steps instead of four K = 16
// ones: there a lane holds A[lane % 16][k = 8 (lane / 16) + i] and B[k = 8
// (lane / 16) + i][lane % 16], i < 8, and the same D layout.  A lane's 8 B
// values are its D values of two consecutive 16-row blocks, so within a K = 32
// step the hidden unit of slot (lane / 16, i) is 16 (2p + i / 4) + 4 (lane /
// 16) + i % 4; the weights are loaded in that order, and the contraction is
// the same sum over all 64 units.  The weight gradients (sums over variables)
// need the activations with the variable index as K; those tiles go through
// LDS.
#include <cmath>

#include <algorithm>
#include <mutex>
#include <string>

#include "pdhg_device.hpp"
#include "pdhg_internal.hpp"
#include "pdhg_mlp.hpp"

namespace pdhg {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short f2bf(float f)
{
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u); // round to nearest, ties to even
    return (short)(u >> 16);
}

__device__ __forceinline__ float bf2f(short b) { return __uint_as_float(((unsigned)(unsigned short)b) << 16); }

__device__ __forceinline__ f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                  0, 0, 0);
}

// hidden unit of K = 32 step p, slot (lane group lg, element i)
__device__ __forceinline__ int k32_unit(int p, int lg, int i) { return 16 * (2 * p + (i >> 2)) + 4 * lg + (i & 3); }

// the B operand of K = 32 step p: the D values of 16-row blocks 2p and 2p + 1
__device__ __forceinline__ bf16x8 k32_pair(const bf16x4 &lo, const bf16x4 &hi)
{
    return bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}

// Four consecutive bfloat16 values in one 8-byte load (the library's own
// weight copies: 256-byte aligned, offsets a multiple of four).
__device__ __forceinline__ bf16x4 load4(const short *__restrict__ p) { return *reinterpret_cast<const bf16x4 *>(p); }

// the A operand of K = 32 step p for weight row `row` of a 64 x 64 matrix: two
// runs of four consecutive units (k32_unit)
__device__ __forceinline__ bf16x8 load_k32(const short *__restrict__ w, int row, int p, int lg)
{
    return k32_pair(load4(w + row * 64 + k32_unit(p, lg, 0)), load4(w + row * 64 + k32_unit(p, lg, 4)));
}

// parameter offsets in the flat vector: w1 (64x16), b1, w2 (64x64), b2, w3, b3
constexpr int OFF_W1 = 0, OFF_B1 = 1024, OFF_W2 = 1088, OFF_B2 = 5184, OFF_W3 = 5248, OFF_B3 = 5312;

struct MlpW {
    const short *w1b, *w2b, *w3b; // bfloat16 copies
    const short *w2tb;            // W2 transposed, bfloat16 (the gradient's backward contraction)
    const float *p;               // float32 master values (biases read from here)
};

// ----------------------------------------------------------------- forward
// The four features 4 lg .. 4 lg + 3 of variable v as the B operand: bfloat16
// ones as they are, float32 ones rounded here.  A caller's buffers are only
// element-aligned, hence the copies (one 8- or 16-byte load each).
__device__ __forceinline__ bf16x4 load_features(const short *__restrict__ F, int64_t v, int lg)
{
    bf16x4 f;
    __builtin_memcpy(&f, F + v * 16 + 4 * lg, sizeof(f));
    return f;
}

__device__ __forceinline__ bf16x4 load_features(const float *__restrict__ F, int64_t v, int lg)
{
    f32x4 f;
    __builtin_memcpy(&f, F + v * 16 + 4 * lg, sizeof(f));
    return bf16x4{f2bf(f[0]), f2bf(f[1]), f2bf(f[2]), f2bf(f[3])};
}

// A wave takes tiles of 16 variables by turns.  A call is bound by its chain of
// loads and matrix steps, so the features, weights and biases go out together,
// as 8- and 16-byte loads; and where there are more workgroups than CUs, by the
// weights, which every wave reads: 32 loads of 16 lines each, more of the CU's
// cache than the features and the arithmetic of a tile (forward_grid).  65,536
// variables, host calls included: 11.9 us per call with a separate bfloat16
// pass and 2-byte weight loads, 9.1-11.2 with one tile a wave, 6.4 with four, on
// the same features again; on features that come from HBM 15.1 -> 7.5.
template <typename FT>
__global__ __launch_bounds__(kBlock) void k_mlp_forward(const FT *__restrict__ F, int64_t N, MlpW w,
                                                       float *__restrict__ logits)
{
    const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    const int64_t ntiles = (N + 15) / 16;
    const int64_t nwaves = (int64_t)gridDim.x * (kBlock / 64);
    int64_t t = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    if (t >= ntiles) return;
    // the first tile's features go out with the weights
    bf16x4 fb = load_features(F, t * 16 + lr < N ? t * 16 + lr : N - 1, lg);
    bf16x4 w1a[4], w3b[4];
    bf16x8 w2a[4][2];
    f32x4 b1[4], b2[4];
#pragma unroll
    for (int mb = 0; mb < 4; mb++) {
        w1a[mb] = load4(w.w1b + (16 * mb + lr) * 16 + 4 * lg);
#pragma unroll
        for (int p = 0; p < 2; p++) w2a[mb][p] = load_k32(w.w2b, 16 * mb + lr, p, lg);
        w3b[mb] = load4(w.w3b + 16 * mb + 4 * lg);
        b1[mb] = *reinterpret_cast<const f32x4 *>(w.p + OFF_B1 + 16 * mb + 4 * lg);
        b2[mb] = *reinterpret_cast<const f32x4 *>(w.p + OFF_B2 + 16 * mb + 4 * lg);
    }
    const float b3 = w.p[OFF_B3];
    for (; t < ntiles; t += nwaves) {
        const int64_t v = t * 16 + lr; // lanes past N work on the last variable and store nothing
        bf16x4 h1b[4];
#pragma unroll
        for (int mb = 0; mb < 4; mb++) {
            const f32x4 a = mfma16(w1a[mb], fb, f32x4{0, 0, 0, 0});
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float h = a[r] + b1[mb][r];
                h1b[mb][r] = f2bf(h > 0.0f ? h : 0.0f);
            }
        }
        const int64_t vn = v + nwaves * 16; // the next tile's features, before this one's second layer
        fb = load_features(F, vn < N ? vn : N - 1, lg);
        float part = 0.0f;
        const bf16x8 h1p[2] = {k32_pair(h1b[0], h1b[1]), k32_pair(h1b[2], h1b[3])};
#pragma unroll
        for (int mb = 0; mb < 4; mb++) {
            f32x4 a = {0, 0, 0, 0};
#pragma unroll
            for (int p = 0; p < 2; p++) a = mfma32(w2a[mb][p], h1p[p], a);
#pragma unroll
            for (int r = 0; r < 4; r++) {
                float hv = a[r] + b2[mb][r];
                hv = hv > 0.0f ? hv : 0.0f;
                part += bf2f(w3b[mb][r]) * hv;
            }
        }
        part += __shfl_xor(part, 16, 64);
        part += __shfl_xor(part, 32, 64);
        if (lg == 0 && v < N) logits[v] = part + b3;
    }
}

// ---------------------------------------------------------------- gradient
// Each wave handles kGradTiles tiles of 16 samples of the minibatch
// (samples idx[b0 + k], k < bsz) and writes its partial gradient (5313
// values) and partial loss; k_mlp_reduce sums the partials in wave order.
// A minibatch of 4,096 samples is only 128 waves and every one a serial chain:
// one wave per workgroup spreads them over 128 CUs instead of 32, both tiles'
// samples are loaded before the weights, and the weights come in 8-byte loads
// (W2^T from a transposed copy): 18.6 -> 13.1 us.
__device__ __forceinline__ float softplus(float x) { return x > 0.0f ? x + log1pf(expf(-x)) : log1pf(expf(x)); }

// sum over each row of 16 lanes, neighbours first, in the row's lowest lane
__device__ __forceinline__ float pair_sum16(float v)
{
    v += lane_up<1>(v);
    v += lane_up<2>(v);
    v += lane_up<4>(v);
    return v + lane_up<8>(v);
}

constexpr int kGradTiles = 2; // tiles of 16 samples per wave

__global__ __launch_bounds__(64) void k_mlp_grad(const short *__restrict__ F, const float *__restrict__ Y,
                                                const int *__restrict__ idx, int64_t b0, int bsz, float pw, MlpW w,
                                                float *__restrict__ part, float *__restrict__ lossp)
{
    __shared__ short a_s[64 * 16];
    __shared__ short b_s[64 * 16];
    __shared__ short f_s[16 * 16];
    const int lane = threadIdx.x, lr = lane & 15, lg = lane >> 4;
    const int gw = blockIdx.x; // wave number: one wave per workgroup
    // every tile's samples before the weights: index, then features and label
    bf16x4 ft[kGradTiles];
    float yt[kGradTiles];
    int rows[kGradTiles];
#pragma unroll
    for (int tt = 0; tt < kGradTiles; tt++) {
        const int k = (gw * kGradTiles + tt) * 16 + lr;
        rows[tt] = idx[b0 + (k < bsz ? k : bsz - 1)];
    }
#pragma unroll
    for (int tt = 0; tt < kGradTiles; tt++) {
        ft[tt] = load4(F + (int64_t)rows[tt] * 16 + 4 * lg);
        yt[tt] = Y[rows[tt]];
    }
    bf16x4 w1a[4], w3b[4];
    bf16x8 w2a[4][2], w2t[4][2];
    f32x4 b1[4], b2[4];
#pragma unroll
    for (int mb = 0; mb < 4; mb++) {
        w1a[mb] = load4(w.w1b + (16 * mb + lr) * 16 + 4 * lg);
#pragma unroll
        for (int p = 0; p < 2; p++) {
            w2a[mb][p] = load_k32(w.w2b, 16 * mb + lr, p, lg);
            w2t[mb][p] = load_k32(w.w2tb, 16 * mb + lr, p, lg); // W2^T
        }
        w3b[mb] = load4(w.w3b + 16 * mb + 4 * lg);
        b1[mb] = *reinterpret_cast<const f32x4 *>(w.p + OFF_B1 + 16 * mb + 4 * lg);
        b2[mb] = *reinterpret_cast<const f32x4 *>(w.p + OFF_B2 + 16 * mb + 4 * lg);
    }
    const float b3 = w.p[OFF_B3];
    const float inv_b = 1.0f / (float)bsz;
    f32x4 gw2[4][4], gw1[4];
    float gb1[4][4], gb2[4][4], gw3[4][4], gb3 = 0.0f, loss = 0.0f;
#pragma unroll
    for (int mb = 0; mb < 4; mb++) {
        gw1[mb] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; r++) gb1[mb][r] = gb2[mb][r] = gw3[mb][r] = 0.0f;
#pragma unroll
        for (int nb = 0; nb < 4; nb++) gw2[mb][nb] = f32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int tt = 0; tt < kGradTiles; tt++) {
        const int k = (gw * kGradTiles + tt) * 16 + lr; // sample slot in the minibatch
        const bool valid = k < bsz;
        const bf16x4 fb = valid ? ft[tt] : bf16x4{0, 0, 0, 0};
        const float y = valid ? yt[tt] : 0.0f;
        // forward, keeping the activations
        float h1[4][4], h2[4][4];
        bf16x4 h1b[4];
#pragma unroll
        for (int mb = 0; mb < 4; mb++) {
            const f32x4 a = mfma16(w1a[mb], fb, f32x4{0, 0, 0, 0});
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float h = a[r] + b1[mb][r];
                h1[mb][r] = h > 0.0f ? h : 0.0f;
                h1b[mb][r] = f2bf(h1[mb][r]);
            }
        }
        float z = 0.0f;
        const bf16x8 h1p[2] = {k32_pair(h1b[0], h1b[1]), k32_pair(h1b[2], h1b[3])};
#pragma unroll
        for (int mb = 0; mb < 4; mb++) {
            f32x4 a = {0, 0, 0, 0};
#pragma unroll
            for (int p = 0; p < 2; p++) a = mfma32(w2a[mb][p], h1p[p], a);
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float hv = a[r] + b2[mb][r];
                h2[mb][r] = hv > 0.0f ? hv : 0.0f;
                z += bf2f(w3b[mb][r]) * h2[mb][r];
            }
        }
        z += __shfl_xor(z, 16, 64);
        z += __shfl_xor(z, 32, 64);
        z += b3;
        // dL/dz of the weighted binary cross-entropy, averaged over the minibatch
        float dz = 0.0f;
        if (valid) {
            const float s = 1.0f / (1.0f + expf(-z));
            dz = (s * (pw * y + 1.0f - y) - pw * y) * inv_b;
            if (lg == 0) {
                loss += pw * y * softplus(-z) + (1.0f - y) * softplus(z);
                gb3 += dz;
            }
        }
        // layer 3 and 2 gradients
        bf16x4 dh2b[4];
#pragma unroll
        for (int mb = 0; mb < 4; mb++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                gw3[mb][r] += dz * h2[mb][r];
                const float d = h2[mb][r] > 0.0f ? dz * bf2f(w3b[mb][r]) : 0.0f;
                gb2[mb][r] += d;
                dh2b[mb][r] = f2bf(d);
            }
        // dH1^T = W2^T dH2^T, masked by relu
        bf16x4 dh1b[4];
        const bf16x8 dh2p[2] = {k32_pair(dh2b[0], dh2b[1]), k32_pair(dh2b[2], dh2b[3])};
#pragma unroll
        for (int mb = 0; mb < 4; mb++) {
            f32x4 a = {0, 0, 0, 0};
#pragma unroll
            for (int p = 0; p < 2; p++) a = mfma32(w2t[mb][p], dh2p[p], a);
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float d = h1[mb][r] > 0.0f ? a[r] : 0.0f;
                gb1[mb][r] += d;
                dh1b[mb][r] = f2bf(d);
            }
        }
        // dW2 += dH2^T H1 : both tiles transposed through LDS (K = samples)
#pragma unroll
        for (int mb = 0; mb < 4; mb++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                a_s[(16 * mb + 4 * lg + r) * 16 + lr] = dh2b[mb][r];
                b_s[(16 * mb + 4 * lg + r) * 16 + lr] = h1b[mb][r];
            }
#pragma unroll
        for (int i = 0; i < 4; i++) f_s[lr * 16 + 4 * lg + i] = fb[i];
        __syncthreads();
        bf16x4 A2[4], B2[4], Bf;
#pragma unroll
        for (int mb = 0; mb < 4; mb++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                A2[mb][i] = a_s[(16 * mb + lr) * 16 + 4 * lg + i];
                B2[mb][i] = b_s[(16 * mb + lr) * 16 + 4 * lg + i];
            }
#pragma unroll
        for (int i = 0; i < 4; i++) Bf[i] = f_s[(4 * lg + i) * 16 + lr];
        __syncthreads();
#pragma unroll
        for (int mb = 0; mb < 4; mb++)
#pragma unroll
            for (int nb = 0; nb < 4; nb++) gw2[mb][nb] = mfma16(A2[mb], B2[nb], gw2[mb][nb]);
        // dW1 += dH1^T F
#pragma unroll
        for (int mb = 0; mb < 4; mb++)
#pragma unroll
            for (int r = 0; r < 4; r++) a_s[(16 * mb + 4 * lg + r) * 16 + lr] = dh1b[mb][r];
        __syncthreads();
#pragma unroll
        for (int mb = 0; mb < 4; mb++) {
            bf16x4 A1;
#pragma unroll
            for (int i = 0; i < 4; i++) A1[i] = a_s[(16 * mb + lr) * 16 + 4 * lg + i];
            gw1[mb] = mfma16(A1, Bf, gw1[mb]);
        }
        __syncthreads();
    }
    // per-wave partial gradient, fixed lane order
    float *out = part + (size_t)gw * MLP_NPARAMS;
#pragma unroll
    for (int mb = 0; mb < 4; mb++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int h = 16 * mb + 4 * lg + r;
            out[OFF_W1 + h * 16 + lr] = gw1[mb][r];
#pragma unroll
            for (int nb = 0; nb < 4; nb++) out[OFF_W2 + h * 64 + 16 * nb + lr] = gw2[mb][nb][r];
            float s1 = gb1[mb][r], s2 = gb2[mb][r], s3 = gw3[mb][r];
            s1 = pair_sum16(s1);
            s2 = pair_sum16(s2);
            s3 = pair_sum16(s3);
            if (lr == 0) {
                out[OFF_B1 + h] = s1;
                out[OFF_B2 + h] = s2;
                out[OFF_W3 + h] = s3;
            }
        }
    gb3 = pair_sum16(gb3);
    loss = pair_sum16(loss);
    gb3 += lane_up<16>(gb3);
    loss += lane_up<16>(loss);
    gb3 += lane_up<32>(gb3);
    loss += lane_up<32>(loss);
    if (lane == 0) {
        out[OFF_B3] = gb3;
        lossp[gw] = loss;
    }
}

// Adam (Kingma and Ba 2015): bc1 = 1 - beta1^t, bc2 = 1 - beta2^t
struct AdamStep {
    float lr, beta1, beta2, eps, bc1, bc2;
};

// the bfloat16 copies of parameter k
__device__ __forceinline__ void store_bf16(int k, float pk, short *__restrict__ w1b, short *__restrict__ w2b,
                                           short *__restrict__ w3b, short *__restrict__ w2tb)
{
    if (k < OFF_B1) w1b[k - OFF_W1] = f2bf(pk);
    else if (k >= OFF_W2 && k < OFF_B2) {
        const int e = k - OFF_W2;
        w2b[e] = f2bf(pk);
        w2tb[(e & 63) * 64 + (e >> 6)] = f2bf(pk);
    } else if (k >= OFF_W3 && k < OFF_B3) w3b[k - OFF_W3] = f2bf(pk);
}

// grad[p] = sum over waves of part[w][p], in wave order, kReduceDepth loads
// in flight; with ADAM the same thread then takes the Adam step on the
// float32 master value and refreshes its bfloat16 copies, so a minibatch is
// two launches.  The workgroup past the parameters adds up the losses, in
// wave order, loaded side by side through LDS.  Measured (minibatch 4,096, 128
// waves): 34.1 us for the sum and 4.5 us for a separate Adam launch before,
// most of it one thread's chain of dependent loss loads.
constexpr int kReduceBlock = 64;
constexpr int kReduceDepth = 32;
constexpr int kLossChunk = 1024;

template <bool ADAM>
__global__ __launch_bounds__(kReduceBlock) void k_mlp_reduce(const float *__restrict__ part, int nw,
                                                            const float *__restrict__ lossp,
                                                            float *__restrict__ grad, double *__restrict__ loss_acc,
                                                            AdamStep ad, float *__restrict__ pv, float *__restrict__ m,
                                                            float *__restrict__ v, short *__restrict__ w1b,
                                                            short *__restrict__ w2b, short *__restrict__ w3b,
                                                            short *__restrict__ w2tb)
{
    __shared__ float s_loss[kLossChunk];
    if (blockIdx.x == gridDim.x - 1) {
        double l = 0.0;
        for (int w0 = 0; w0 < nw; w0 += kLossChunk) {
            const int len = nw - w0 < kLossChunk ? nw - w0 : kLossChunk;
            for (int k = threadIdx.x; k < len; k += kReduceBlock) s_loss[k] = lossp[w0 + k];
            __syncthreads();
            if (threadIdx.x == 0)
                for (int k = 0; k < len; k++) l += (double)s_loss[k];
            __syncthreads();
        }
        if (threadIdx.x == 0) loss_acc[0] += l;
        return;
    }
    const int p = blockIdx.x * kReduceBlock + threadIdx.x;
    if (p >= MLP_NPARAMS) return;
    float acc = 0.0f;
    int w = 0;
    for (; w + kReduceDepth <= nw; w += kReduceDepth) {
        float a[kReduceDepth];
#pragma unroll
        for (int u = 0; u < kReduceDepth; u++) a[u] = part[(size_t)(w + u) * MLP_NPARAMS + p];
#pragma unroll
        for (int u = 0; u < kReduceDepth; u++) acc += a[u];
    }
    for (; w < nw; w++) acc += part[(size_t)w * MLP_NPARAMS + p];
    if (!ADAM) {
        grad[p] = acc;
        return;
    }
    const float mk = ad.beta1 * m[p] + (1.0f - ad.beta1) * acc;
    const float vk = ad.beta2 * v[p] + (1.0f - ad.beta2) * acc * acc;
    m[p] = mk;
    v[p] = vk;
    const float pk = pv[p] - ad.lr * (mk / ad.bc1) / (sqrtf(vk / ad.bc2) + ad.eps);
    pv[p] = pk;
    store_bf16(p, pk, w1b, w2b, w3b, w2tb);
}

// bfloat16 copies of the weights from the master values
__global__ __launch_bounds__(kBlock) void k_mlp_sync_bf16(const float *__restrict__ p, short *__restrict__ w1b,
                                                         short *__restrict__ w2b, short *__restrict__ w3b,
                                                         short *__restrict__ w2tb)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k < MLP_NPARAMS) store_bf16(k, p[k], w1b, w2b, w3b, w2tb);
}

// float32 features (N x 16) to bfloat16
__global__ __launch_bounds__(kBlock) void k_to_bf16(int64_t len, const float *__restrict__ src, short *__restrict__ dst)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < len; i += (int64_t)gridDim.x * kBlock)
        dst[i] = f2bf(src[i]);
}

// Kaiming-uniform weights, bound sqrt(6 / fan_in), from splitmix64 of a
// counter (padding columns of W1 stay 0); zero biases; zero Adam state
__device__ __forceinline__ uint64_t mix64(uint64_t x)
{
    uint64_t z = x + 0x9E3779B97F4A7C15ULL;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(kBlock) void k_mlp_init(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                                                    uint64_t seed)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= MLP_NPARAMS) return;
    const double u = (double)(mix64(seed ^ ((uint64_t)k * 0x9E3779B97F4A7C15ULL)) >> 11) * (1.0 / 9007199254740992.0);
    float val = 0.0f;
    if (k < OFF_B1) val = ((k % 16) < 12) ? (float)((2.0 * u - 1.0) * sqrt(6.0 / 12.0)) : 0.0f;
    else if (k >= OFF_W2 && k < OFF_B2) val = (float)((2.0 * u - 1.0) * sqrt(6.0 / 64.0));
    else if (k >= OFF_W3 && k < OFF_B3) val = (float)((2.0 * u - 1.0) * sqrt(6.0 / 64.0));
    p[k] = val;
    m[k] = 0.0f;
    v[k] = 0.0f;
}

hipError_t mlp_init(pdhg_mlp *net, uint64_t seed)
{
    // on the pass stream, so that its first launch, which sets it up, is not a caller's
    hipLaunchKernelGGL(k_mlp_init, dim3((MLP_NPARAMS + kBlock - 1) / kBlock), dim3(kBlock), 0, net->pass, net->p, net->m,
                       net->v, seed);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = mlp_sync(net, net->pass);
    return e == hipSuccess ? hipStreamSynchronize(net->pass) : e;
}

static MlpW weights(const pdhg_mlp *net) { return MlpW{net->w1b, net->w2b, net->w3b, net->w2tb, net->p}; }

hipError_t mlp_sync(pdhg_mlp *net, hipStream_t st)
{
    hipLaunchKernelGGL(k_mlp_sync_bf16, dim3((MLP_NPARAMS + kBlock - 1) / kBlock), dim3(kBlock), 0, st, net->p,
                       net->w1b, net->w2b, net->w3b, net->w2tb);
    return hipGetLastError();
}

hipError_t mlp_features_to_bf16(hipStream_t st, const float *src, short *dst, int64_t n_rows)
{
    hipLaunchKernelGGL(k_to_bf16, dim3(grid_for(n_rows * 16, kBlock, 65536)), dim3(kBlock), 0, st, n_rows * 16, src, dst);
    return hipGetLastError();
}

// Workgroups of a forward pass: one tile a wave until every CU has a workgroup,
// then as many tiles a wave as keep it at one, at most 8 (16 past a million
// variables, where the chain of a wave's tiles hides behind the other waves).
// us by rocprofv3 on the same features again, one tile a wave -> this rule: 65,536 variables 11.4 -> 6.0,
// 131,072 20.8 -> 8.9 (9.2 with 4 tiles, 13.5 with 16), 262,144 39.8 -> 13.0
// (15.1, 14.3), 1,048,576 152 -> 34 (38 with 8), 4,194,304 598 -> 108 (126).
static int forward_grid(int64_t tiles)
{
    const int64_t full = (tiles + 3) / 4; // one tile a wave
    const int64_t most = full < 16384 ? 8 : 16, per = std::min(most, (full + 255) / 256);
    return grid_for((full + per - 1) / per, 1, 1 << 20);
}

template <typename FT>
static hipError_t forward_impl(const pdhg_mlp *net, hipStream_t st, const FT *F, int64_t N, float *logits)
{
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_mlp_forward<FT>), dim3(forward_grid((N + 15) / 16)), dim3(kBlock), 0, st, F, N, weights(net), logits);
    return hipGetLastError();
}

hipError_t mlp_forward(const pdhg_mlp *net, hipStream_t st, const short *F, int64_t N, float *logits)
{
    return forward_impl(net, st, F, N, logits);
}

// one minibatch: gradient into net->grad (adam NULL) or an Adam step with it,
// loss added to net->loss_acc
static hipError_t grad_impl(pdhg_mlp *net, const short *F, const float *Y, const int *idx, int64_t b0, int bsz, float pw,
                            const AdamStep *adam)
{
    const int tiles = (bsz + 15) / 16;
    const int nw = (tiles + kGradTiles - 1) / kGradTiles;
    if (nw > net->max_waves) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mlp_grad, dim3(nw), dim3(64), 0, net->stream, F, Y, idx, b0, bsz, pw, weights(net), net->part,
                       net->lossp);
    const dim3 grid((MLP_NPARAMS + kReduceBlock - 1) / kReduceBlock + 1);
    if (adam)
        hipLaunchKernelGGL((k_mlp_reduce<true>), grid, dim3(kReduceBlock), 0, net->stream, net->part, nw, net->lossp,
                           net->grad, net->loss_acc, *adam, net->p, net->m, net->v, net->w1b, net->w2b, net->w3b,
                           net->w2tb);
    else
        hipLaunchKernelGGL((k_mlp_reduce<false>), grid, dim3(kReduceBlock), 0, net->stream, net->part, nw, net->lossp,
                           net->grad, net->loss_acc, AdamStep{}, net->p, net->m, net->v, net->w1b, net->w2b, net->w3b,
                           net->w2tb);
    return hipGetLastError();
}

hipError_t mlp_grad(pdhg_mlp *net, const short *F, const float *Y, const int *idx, int64_t b0, int bsz, float pw)
{
    return grad_impl(net, F, Y, idx, b0, bsz, pw, nullptr);
}

hipError_t mlp_train_step(pdhg_mlp *net, const short *F, const float *Y, const int *idx, int64_t b0, int bsz, float pw,
                          float lr, float beta1, float beta2, float eps, int64_t t)
{
    const AdamStep ad{lr, beta1, beta2, eps, 1.0f - powf(beta1, (float)t), 1.0f - powf(beta2, (float)t)};
    return grad_impl(net, F, Y, idx, b0, bsz, pw, &ad);
}

} // namespace pdhg

// ------------------------------------------------- forward without allocation
// For callers that cannot allocate (graph capture, serving loops): the
// kernel reads the caller's float32 features and rounds them in registers
// (the same values as a bfloat16 copy, one launch instead of two).  Only
// where the logits overlap the features, which are then overwritten while
// other waves still read, a bfloat16 copy is staged first; it lives in this
// file-scope device array instead of a buffer allocated per call.  Every GPU the library runs
// on holds its own copy until the process ends.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in symbol): the
// device address comes from hipGetSymbolAddress, once per device with that
// device current, and is kept per device.
namespace pdhg {
namespace {

constexpr int64_t kNoAllocMaxRows = 65536;     // variables per call
constexpr int kMaxDevices = 64;
static __device__ __align__(256) short scratch[16 * kNoAllocMaxRows]; // 2 MiB
short *g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;

// the current device's address of `scratch` (looked up on first use)
hipError_t scratch_for_current_device(short **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = (short *)p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

} // namespace

hipError_t mlp_scratch_setup() // at pdhg_mlp_create, on the device the network lives on
{
    short *p = nullptr;
    return scratch_for_current_device(&p);
}

// Forward passes of callers who name no stream run in the order of their calls
// on a device: such a caller may hand a buffer that one network's pass still
// writes to the next network's pass.  The networks of a device share one stream
// for them, made with the first and given back with the last (a stream per
// network with events between them measured 21 us per call by turns, one
// stream 5.6).  What works on a network's own stream waits for its passes first;
// those that another thread calls meanwhile are enqueued on that stream, between
// a training's steps, and ordered with the shared one by events.
namespace {
struct PassStream {
    hipStream_t st = nullptr;
    int users = 0;
};
std::mutex g_pass_mu;
PassStream g_pass[kMaxDevices];
} // namespace

hipError_t mlp_pass_open(pdhg_mlp *net)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_pass_mu);
    PassStream &p = g_pass[dev];
    if (!p.st && (e = hipStreamCreate(&p.st)) != hipSuccess) return e;
    p.users++;
    net->device = dev;
    net->pass = p.st;
    return hipSuccess;
}

void mlp_pass_close(pdhg_mlp *net)
{
    for (hipEvent_t &v : net->order)
        if (v) (void)hipEventDestroy(v);
    if (!net->pass) return;
    std::lock_guard<std::mutex> lock(g_pass_mu);
    PassStream &p = g_pass[net->device];
    net->pass = nullptr;
    if (--p.users > 0) return;
    (void)hipStreamDestroy(p.st);
    p.st = nullptr;
}

hipError_t mlp_stream_open(pdhg_mlp *net)
{
    if (net->stream) return hipSuccess;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev), e2 = hipSuccess;
    if (e == hipSuccess && dev != net->device) e = hipSetDevice(net->device);
    for (hipEvent_t &v : net->order)
        if (e == hipSuccess && !v) e = hipEventCreateWithFlags(&v, hipEventDisableTiming);
    if (e == hipSuccess) e = hipStreamCreate(&net->stream);
    if (dev >= 0 && dev != net->device) e2 = hipSetDevice(dev);
    return e != hipSuccess ? e : e2;
}

hipError_t mlp_pass_wait(pdhg_mlp *net)
{
    if (!net->pass || !net->passed) return hipSuccess;
    net->passed = false;
    return hipStreamSynchronize(net->pass);
}

namespace {
// the pass itself: features and logits on the current device
hipError_t enqueue_pass(pdhg_mlp *net, hipStream_t st, const float *features, int64_t n, float *logits)
{
    const uintptr_t f0 = (uintptr_t)features, f1 = (uintptr_t)(features + 16 * n), l0 = (uintptr_t)logits,
                    l1 = (uintptr_t)(logits + n);
    if (l0 >= f1 || f0 >= l1) return forward_impl(net, st, features, n, logits);
    short *fb = nullptr;
    hipError_t e = scratch_for_current_device(&fb);
    if (e == hipSuccess) e = mlp_features_to_bf16(st, features, fb, n); // every staged row is overwritten: nothing to clear
    return e == hipSuccess ? mlp_forward(net, st, fb, n, logits) : e;
}
} // namespace

} // namespace pdhg

extern "C" int pdhg_mlp_forward_noalloc(pdhg_mlp *net, const float *features, int64_t n, float *logits, void *stream)
{
    using namespace pdhg;
    if (!net || n < 0 || (n > 0 && (!features || !logits)))
        return fail(PDHG_ERR_INVALID_ARG, "bad arguments (NULL network or device pointer, or n < 0)");
    if (n > kNoAllocMaxRows)
        return fail(PDHG_ERR_INVALID_ARG, "pdhg_mlp_forward_noalloc takes at most 65536 variables per call");
    if (n == 0) return PDHG_OK;
    hipError_t e = hipSuccess;
    if (stream) {
        e = enqueue_pass(net, (hipStream_t)stream, features, n, logits);
    } else {
        std::lock_guard<std::mutex> lock(net->mu);
        const bool beside = net->busy > 0;
        if (beside) {
            e = hipEventRecord(net->order[0], net->pass);
            if (e == hipSuccess) e = hipStreamWaitEvent(net->stream, net->order[0], 0);
        }
        if (e == hipSuccess) e = enqueue_pass(net, beside ? net->stream : net->pass, features, n, logits);
        if (beside && e == hipSuccess) {
            e = hipEventRecord(net->order[1], net->stream);
            if (e == hipSuccess) e = hipStreamWaitEvent(net->pass, net->order[1], 0);
        }
        net->passed = true;
        net->beside = net->beside || beside;
    }
    if (e != hipSuccess) return fail(PDHG_ERR_HIP, std::string("HIP error in the forward pass: ") + hipGetErrorString(e));
    return PDHG_OK;
}
