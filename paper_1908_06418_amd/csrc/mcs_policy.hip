// Learned branching policy: a 16 -> 64 -> 64 -> 1 ReLU network that scores a
// candidate vertex at a search node.  The search uses the scores to choose v
// within the selected class and the order of its partners w; it never prunes
// on them, so answers are unchanged (the paper's Solve explores or bounds
// every child regardless of order).
//
// Parameters are float32 "master" values packed as W1[64][16], b1[64],
// W2[64][64], b2[64], w3[64], b3.  Inputs are half precision.  Every multiply
// uses the half-rounded weights with float32 accumulation -- the same
// arithmetic the search applies at inference (mcs_policy_score).
//
// The contractions run on the matrix cores, with tiles of 32 rows held
// "unit by row": the columns of a result tile are rows of the batch, so lane
// l keeps row l % 32 through the whole network and its 16 registers are 16
// hidden units (acc_unit).  A result tile is then the next product's right
// operand as it stands: the order in which a contraction takes its units is
// free as long as the weights are laid out to match.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mcs_policy.h"

namespace mcs {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef v8h v8h_a2 __attribute__((aligned(2)));  // (rows of the caller's: any half)
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float round_half(float x) { return __half2float(__float2half(x)); }

// Hidden unit of register r of a 32 x 32 result tile in a lane of half `hi`
// (lanes 32..63): units 4 * hi .. 4 * hi + 3 of every eight.
__device__ __forceinline__ constexpr int acc_unit(int r, int hi) {
    return 8 * (r >> 2) + 4 * hi + (r & 3);
}

// Layer 1 of 32 rows: units 32 * m .. + 31.  Half inputs and half weights,
// exact products, float32 sums: one 32x32x16 product.
__device__ __forceinline__ v16f layer1(const v8h &w1, const v8h &x, const v16f &b1) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(w1, x, b1, 0, 0, 0);
}
// Its left operand: lane l holds unit 32 m + l % 32, features 8 (l / 32) .. + 7.
__device__ __forceinline__ v8h load_w1(const float *P, int m, int lo, int hi) {
    v8h w;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        w[i] = (_Float16)P[kOffW1 + (32 * m + lo) * kPolicyF + 8 * hi + i];
    return w;
}
// A row's features as the right operand (zeros past the last row).
__device__ __forceinline__ v8h load_x(const uint16_t *X, int row, int rows, int hi) {
    v8h x = {};
    if (row < rows)
        x = *(const v8h_a2 *)(X + (size_t)row * kPolicyF + 8 * hi);
    return x;
}
// The half-rounded bias (or output weight) of each register's unit.
__device__ __forceinline__ v16f load_units(const float *p, int m, int hi) {
    v16f v;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        v[r] = round_half(p[32 * m + acc_unit(r, hi)]);
    return v;
}
// The other half-wavefront's x (lane l from lane l ^ 32).
__device__ __forceinline__ float other_half(float x) { return __shfl_xor(x, 32, 64); }

// Layer 2, units 32 m .. + 31, from float32 activations on float32 matrix
// instructions; W2 (half-rounded floats) at w2, rows ld apart.
__device__ __forceinline__ v16f layer2_f32(const float *w2, int ld, const v16f h[2], int m, int lo,
                                           int hi, v16f acc) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(
                w2[(32 * m + lo) * ld + 32 * c + acc_unit(r, hi)], h[c][r], acc, 0, 0, 0);
    return acc;
}

// Scores.  Layer 2's activations are float32, its weights half precision; on
// float32 matrix instructions the layer would take twice the time of the rest,
// so each activation is cut into three half-precision numbers, h = a + b 2^-11
// + c 2^-22: a = half(h) leaves at most 2^-11 |h|, b at most 2^-22 |h|, and c
// the last bits of h's 24.  Nothing is left out: a tile with an activation of
// which something would be (beyond the half range, or with bits below 2^-46)
// takes the float32 instructions, and so does every tile where a weight of the
// layer rounds to infinity (its product with a piece that is zero would be no
// number).  The products of a have accumulators of their own, those of b and c
// others.  Bound by the vector work around the products (cutting the activations, w3).
// 1,000,000 rows: 45 us a call (229 TFLOP/s) against 1,952 us with one row per
// lane and float32 FMAs (5.3); with two pieces, which leave out up to 2^-23 |h|
// and more below 2^-14, it was 31.
__global__ void __launch_bounds__(256, 2) policy_forward_kernel(const uint16_t *X, int rows,
                                                                const float *P, float *logits) {
    __shared__ float s2[kPolicyH * (kPolicyH + 1)];  // W2, for tiles out of the half range
    __shared__ float s3[3 * kPolicyH];               // b2, w3, b1
    const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5;
    for (int i = threadIdx.x; i < kPolicyH * kPolicyH; i += blockDim.x)
        s2[(i / kPolicyH) * (kPolicyH + 1) + i % kPolicyH] = round_half(P[kOffW2 + i]);
    for (int i = threadIdx.x; i < kPolicyH; i += blockDim.x) {
        s3[i] = round_half(P[kOffB2 + i]);
        s3[kPolicyH + i] = round_half(P[kOffW3 + i]);
        s3[2 * kPolicyH + i] = round_half(P[kOffB1 + i]);
    }
    __syncthreads();
    v8h w1[2], w2[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        w1[m] = load_w1(P, m, lo, hi);
        // chunk c contracts units 16 c .. + 15, in the order in which the
        // two half-wavefronts hold them
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w2[m][c][i] = (_Float16)s2[(32 * m + lo) * (kPolicyH + 1) + 32 * (c >> 1) +
                                           acc_unit(8 * (c & 1) + i, hi)];
    }
    const float b3 = round_half(P[kOffB3]);
    float sum2 = 0.f;  // 0, or NaN if a weight of layer 2 is no finite number
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                sum2 += 0.f * (float)w2[m][c][i];
    const bool finite = __ballot(sum2 != 0.f) == 0;
    const int tiles = (rows + 31) / 32, step = gridDim.x * (blockDim.x >> 6);
    for (int tile = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); tile < tiles;
         tile += step) {
        const int row = 32 * tile + lo;
        const v8h x = load_x(X, row, rows, hi);
        asm volatile("" ::: "memory");  // (b1, b2 and w3 stay in LDS between tiles)
        v16f h[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            v16f b1;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                b1[r] = s3[2 * kPolicyH + 32 * m + acc_unit(r, hi)];
            h[m] = layer1(w1[m], x, b1);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                h[m][r] = fmaxf(h[m][r], 0.f);
        }
        float z = 0.f;
        v8h a[4], b[4], c[4];
        uint32_t left = 0;  // not 0: some activation is more than its pieces
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float v = h[q >> 1][8 * (q & 1) + i];
                a[q][i] = (_Float16)v;
                const float vb = (v - (float)a[q][i]) * 2048.f;
                b[q][i] = (_Float16)vb;
                const float vc = (vb - (float)b[q][i]) * 2048.f;
                c[q][i] = (_Float16)vc;
                left |= __float_as_uint(vc - (float)c[q][i]);
            }
        if (finite && __ballot(left != 0) == 0) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                v16f acc, low = {};
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[r] = s3[32 * m + acc_unit(r, hi)];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    low = __builtin_amdgcn_mfma_f32_32x32x16_f16(w2[m][q], c[q], low, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    low[r] *= 1.f / 2048.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(w2[m][q], a[q], acc, 0, 0, 0);
                    low = __builtin_amdgcn_mfma_f32_32x32x16_f16(w2[m][q], b[q], low, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    z = fmaf(s3[kPolicyH + 32 * m + acc_unit(r, hi)],
                             fmaxf(fmaf(low[r], 1.f / 2048.f, acc[r]), 0.f), z);
            }
        } else {
            for (int m = 0; m < 2; ++m) {
                v16f acc;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[r] = s3[32 * m + acc_unit(r, hi)];
                acc = layer2_f32(s2, kPolicyH + 1, h, m, lo, hi, acc);
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    z = fmaf(s3[kPolicyH + 32 * m + acc_unit(r, hi)], fmaxf(acc[r], 0.f), z);
            }
        }
        z += other_half(z);
        if (hi == 0 && row < rows)
            logits[row] = z + b3;
    }
}

// LDS of the gradient kernel, in floats: W2 (rows of 65), then for each
// wavefront two unit-by-row tiles of 64 x 33 and the rows' features (32 x
// 17).  The block's sums take the wavefronts' part once they are done.
constexpr int kLdW2 = kPolicyH + 1, kLdT = 33, kLdX = 17;
constexpr int kTile = kPolicyH * kLdT;
constexpr int kWaveLds = 2 * kTile + 32 * kLdX;
constexpr int kGradWaves = 4;
constexpr int kGradLds = kPolicyH * kLdW2 + kGradWaves * kWaveLds;
static_assert(kGradWaves * kWaveLds >= kPolicyParams + 1, "the block's sums fit");

// LDS traffic between lanes of one wavefront keeps its order.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The gradient of the mean binary cross-entropy (already divided by the row
// count) and the summed loss, over the rows of one block's tiles:
// partials[block][kPolicyParams + 1].  All products of float32 values run on
// the float32 matrix instructions.  A wavefront takes tiles of 32 rows and
// keeps its sums of all parameters in registers: W2's gradient as four 32 x
// 32 tiles contracted over the rows, W1's and b1's as two (16 features, a
// column of ones), b2's and w3's per lane.  Only the operands contracted over
// rows go through LDS, to turn units into lanes.  The wavefronts then add
// their sums in order, so the result does not depend on timing.  Gradient and
// update of 41,358 rows, as called from Python: 62 us against 464 us with
// float32 FMAs and one partial per 64 rows (646 of them, added one after
// another); most of what is left is launches.
__global__ void __launch_bounds__(64 * kGradWaves, 1) policy_partial_kernel(
    const uint16_t *X, const float *y, int rows, const float *P, float *partials) {
    __shared__ float s[kGradLds];
    const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5, wv = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < kPolicyH * kPolicyH; i += blockDim.x)
        s[(i / kPolicyH) * kLdW2 + i % kPolicyH] = round_half(P[kOffW2 + i]);
    __syncthreads();
    const float *W2 = s;
    float *sh = s + kPolicyH * kLdW2 + wv * kWaveLds;  // h1 by unit and row
    float *sd = sh + kTile;                            // d2, then d1
    float *sx = sd + kTile;                            // features by row
    v8h w1[2];
    v16f b1[2], b2[2], w3[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        w1[m] = load_w1(P, m, lo, hi);
        b1[m] = load_units(P + kOffB1, m, hi);
        b2[m] = load_units(P + kOffB2, m, hi);
        w3[m] = load_units(P + kOffW3, m, hi);
    }
    const float b3 = round_half(P[kOffB3]);
    v16f gW2[2][2] = {}, gW1[2] = {}, gb2[2] = {}, gw3[2] = {};
    float gb3 = 0.f, loss = 0.f;
    const int tiles = (rows + 31) / 32, step = gridDim.x * kGradWaves;
    for (int tile = blockIdx.x * kGradWaves + wv; tile < tiles; tile += step) {
        const int row = 32 * tile + lo;
        const bool live = row < rows;
        const v8h x = load_x(X, row, rows, hi);
        wave_order();  // the tile before has been read
#pragma unroll
        for (int i = 0; i < 8; ++i)
            sx[lo * kLdX + 8 * hi + i] = (float)x[i];
        v16f h[2], d1[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            h[m] = layer1(w1[m], x, b1[m]);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                h[m][r] = fmaxf(h[m][r], 0.f);
                sh[(32 * m + acc_unit(r, hi)) * kLdT + lo] = h[m][r];
            }
        }
        v16f a2[2];
        float z = 0.f;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            a2[m] = layer2_f32(W2, kLdW2, h, m, lo, hi, b2[m]);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                z = fmaf(w3[m][r], fmaxf(a2[m][r], 0.f), z);
        }
        z += other_half(z);
        z += b3;
        const float yy = live ? y[row] : 0.f;
        // stable form of the binary cross-entropy of sigmoid(z) against y
        const float l = fmaxf(z, 0.f) - z * yy + log1pf(__expf(-fabsf(z)));
        const float sig = 1.f / (1.f + __expf(-z));
        const float dz = live ? (sig - yy) / (float)rows : 0.f;
        if (hi == 0) {
            gb3 += dz;
            loss += live ? l : 0.f;
        }
        // a2 becomes dL/da2
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                gw3[m][r] = live ? fmaf(dz, fmaxf(a2[m][r], 0.f), gw3[m][r]) : gw3[m][r];
                a2[m][r] = a2[m][r] > 0.f ? dz * w3[m][r] : 0.f;
                gb2[m][r] += a2[m][r];
                sd[(32 * m + acc_unit(r, hi)) * kLdT + lo] = a2[m][r];
            }
        wave_order();
        // gW2[u][k] += sum over rows of d2[u] h1[k]
#pragma unroll 4
        for (int q = 0; q < 16; ++q) {
            const int c = 2 * q + hi;  // row of the tile
            const float d0 = sd[lo * kLdT + c], d32 = sd[(32 + lo) * kLdT + c];
            const float h0 = sh[lo * kLdT + c], h32 = sh[(32 + lo) * kLdT + c];
            gW2[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(d0, h0, gW2[0][0], 0, 0, 0);
            gW2[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(d0, h32, gW2[0][1], 0, 0, 0);
            gW2[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(d32, h0, gW2[1][0], 0, 0, 0);
            gW2[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(d32, h32, gW2[1][1], 0, 0, 0);
        }
        // dL/da1 = W2^T d2 where h1 > 0
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            v16f acc = {};
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(
                        W2[(32 * c + acc_unit(r, hi)) * kLdW2 + 32 * m + lo], a2[c][r], acc, 0, 0,
                        0);
            d1[m] = acc;
        }
        wave_order();  // d2 has been read
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                sd[(32 * m + acc_unit(r, hi)) * kLdT + lo] = h[m][r] > 0.f ? d1[m][r] : 0.f;
        wave_order();
        // gW1[u][f] += sum over rows of d1[u] x[f]; column 16: a one, for b1
#pragma unroll 4
        for (int q = 0; q < 16; ++q) {
            const int c = 2 * q + hi;
            const float xf = lo < kPolicyF ? sx[c * kLdX + lo] : lo == kPolicyF ? 1.f : 0.f;
            gW1[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(sd[lo * kLdT + c], xf, gW1[0], 0, 0, 0);
            gW1[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(sd[(32 + lo) * kLdT + c], xf, gW1[1], 0,
                                                          0, 0);
        }
    }
    // sums over the rows (lanes) of what was kept per lane
#pragma unroll
    for (int k = 16; k >= 1; k >>= 1) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                gb2[m][r] += __shfl_xor(gb2[m][r], k, 64);
                gw3[m][r] += __shfl_xor(gw3[m][r], k, 64);
            }
        gb3 += __shfl_xor(gb3, k, 64);
        loss += __shfl_xor(loss, k, 64);
    }
    float *sum = s + kPolicyH * kLdW2;
    __syncthreads();
    for (int i = threadIdx.x; i <= kPolicyParams; i += blockDim.x)
        sum[i] = 0.f;
    for (int w = 0; w < kGradWaves; ++w) {
        __syncthreads();
        if (wv != w)
            continue;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int u = 32 * m + acc_unit(r, hi);
#pragma unroll
                for (int n = 0; n < 2; ++n)
                    sum[kOffW2 + u * kPolicyH + 32 * n + lo] += gW2[m][n][r];
                if (lo < kPolicyF)
                    sum[kOffW1 + u * kPolicyF + lo] += gW1[m][r];
                else if (lo == kPolicyF)
                    sum[kOffB1 + u] += gW1[m][r];
                if (lo == 0) {
                    sum[kOffB2 + u] += gb2[m][r];
                    sum[kOffW3 + u] += gw3[m][r];
                }
            }
        if (lane == 0) {
            sum[kOffB3] += gb3;
            sum[kPolicyParams] += loss;
        }
    }
    __syncthreads();
    float *out = partials + (size_t)blockIdx.x * (kPolicyParams + 1);
    for (int i = threadIdx.x; i <= kPolicyParams; i += blockDim.x)
        out[i] = sum[i];
}

// grads[i] = sum over blocks; loss = summed loss / rows.  Fixed order: 16
// groups of a block take every 16th partial, then the groups are added.
__global__ void __launch_bounds__(1024) policy_reduce_kernel(const float *partials, int blocks,
                                                             int rows, float *grads, float *loss) {
    __shared__ float s[16][64];
    const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + c;
    float acc = 0.f;
    if (i <= kPolicyParams)
#pragma unroll 4
        for (int b = g; b < blocks; b += 16)
            acc += partials[(size_t)b * (kPolicyParams + 1) + i];
    s[g][c] = acc;
    __syncthreads();
    if (g != 0 || i > kPolicyParams)
        return;
    for (int k = 1; k < 16; ++k)
        acc += s[k][c];
    if (i < kPolicyParams)
        grads[i] = acc;
    else if (loss)
        *loss = acc / (float)rows;
}

__global__ void __launch_bounds__(256) policy_sgd_kernel(float *P, const float *G, float lr) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kPolicyParams)
        P[i] -= lr * G[i];
}

__global__ void __launch_bounds__(256) policy_pack_half_kernel(const float *P, uint16_t *H) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kPolicyParams)
        H[i] = __half_as_ushort(__float2half(P[i]));
}

}  // namespace mcs

// ---- C ABI (declared in include/mcs.h) -------------------------------------

#include "mcs.h"

#include <algorithm>

namespace {
mcs_status launch_status(hipError_t e) { return e == hipSuccess ? MCS_OK : MCS_E_DEVICE; }
}  // namespace

extern "C" {

int32_t mcs_policy_param_count(void) { return mcs::kPolicyParams; }

size_t mcs_policy_workspace_size(int32_t rows) {
    if (rows <= 0)
        return 0;
    size_t blocks = ((size_t)rows + 63) / 64;
    return blocks * (mcs::kPolicyParams + 1) * sizeof(float);
}

mcs_status mcs_policy_forward(const uint16_t *x, int32_t rows, const float *params, float *logits,
                              void *stream) {
    if (rows < 0 || (rows > 0 && (!x || !params || !logits)))
        return MCS_E_INVALID;
    if (rows == 0)
        return MCS_OK;
    // (two blocks of four wavefronts stay resident on a CU; each wavefront
    // loads the weights once and then takes every so many tiles of 32 rows)
    hipLaunchKernelGGL(mcs::policy_forward_kernel, dim3(std::min((rows + 127) / 128, 512)),
                       dim3(256), 0, (hipStream_t)stream, x, rows, params, logits);
    return launch_status(hipGetLastError());
}

mcs_status mcs_policy_grad(const uint16_t *x, const float *y, int32_t rows, const float *params,
                           float *grads, float *loss, void *workspace, size_t bytes,
                           void *stream) {
    if (rows <= 0 || !x || !y || !params || !grads)
        return MCS_E_INVALID;
    if (!workspace || bytes < mcs_policy_workspace_size(rows))
        return MCS_E_WORKSPACE;
    // one block per CU at most (and no more than the workspace has room
    // for: one partial per 64 rows)
    const int blocks = std::min((rows + 32 * mcs::kGradWaves - 1) / (32 * mcs::kGradWaves), 256);
    hipStream_t s = (hipStream_t)stream;
    float *partials = (float *)workspace;
    hipLaunchKernelGGL(mcs::policy_partial_kernel, dim3(blocks), dim3(64 * mcs::kGradWaves), 0, s,
                       x, y, rows, params, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return MCS_E_DEVICE;
    hipLaunchKernelGGL(mcs::policy_reduce_kernel, dim3((mcs::kPolicyParams + 64) / 64),
                       dim3(1024), 0, s, partials, blocks, rows, grads, loss);
    return launch_status(hipGetLastError());
}

mcs_status mcs_policy_sgd(float *params, const float *grads, float lr, void *stream) {
    if (!params || !grads)
        return MCS_E_INVALID;
    hipLaunchKernelGGL(mcs::policy_sgd_kernel, dim3((mcs::kPolicyParams + 255) / 256), dim3(256),
                       0, (hipStream_t)stream, params, grads, lr);
    return launch_status(hipGetLastError());
}

mcs_status mcs_policy_pack_half(const float *params, uint16_t *half_params, void *stream) {
    if (!params || !half_params)
        return MCS_E_INVALID;
    hipLaunchKernelGGL(mcs::policy_pack_half_kernel, dim3((mcs::kPolicyParams + 255) / 256),
                       dim3(256), 0, (hipStream_t)stream, params, half_params);
    return launch_status(hipGetLastError());
}

}  // extern "C"
