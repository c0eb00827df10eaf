// Learned warm start for the Newmark solve: a per-edge 4 -> 64 -> 64 -> 1 ReLU network on
// gfx950 matrix cores.  Layer 2 (64 x 64) runs as v_mfma_f32_16x16x32_bf16 tiles (BF16
// operands, FP32 accumulation); layer 1 (K = 4) is computed on the vector ALUs straight
// into the MFMA operand layout; layer 3 is a 64-wide dot reduced across lanes.  Training
// uses the same tiles for the backward products dW2 = dZ2^T H1 (reduction over the batch
// rows, staged through LDS) and dH1 = dZ2 W2 (from registers); Adam keeps FP32 masters.
//
// Operand layout of v_mfma_f32_16x16x32_bf16 (wave64), lane l, g = l / 16:
//   A (16 x 32):  row l % 16, 8 consecutive k starting at 8 g
//   B (32 x 16):  column l % 16, the same 8 k
//   D (16 x 16):  rows 4 g + i (i = 0..3), column l % 16
// Only the pairing of A's and B's k entries within a lane matters for the sum, and both
// operands are always built with the same k order.
#include <algorithm>

#include "fepic_internal.h"

namespace fepic {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kH = 64;           // hidden width
constexpr int kIn = 4;           // inputs per edge
// flat parameter layout: W1[64][4], b1[64], W2[64][64], b2[64], W3[64], b3
constexpr int oW1 = 0, ob1 = 256, oW2 = 320, ob2 = 4416, oW3 = 4480, ob3 = 4544, kNP = 4545;
static_assert(kNP == FEPIC_MLP_N_PARAMS, "parameter layout");

constexpr int kMlpBlock = 256;   // 4 waves

__device__ __forceinline__ floatx4 mfma(const bf16x8& a, const bf16x8& b, const floatx4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

struct MlpLds {
    float W1[kH * kIn];
    float b1[kH], b2[kH], W3[kH];
    float b3;
    alignas(16) __bf16 W2[kH * kH];    // [n][k]
};

__device__ __forceinline__ void load_params(MlpLds& L, const float* __restrict__ P) {
    for (int i = threadIdx.x; i < kH * kIn; i += blockDim.x) L.W1[i] = P[oW1 + i];
    for (int i = threadIdx.x; i < kH; i += blockDim.x) {
        L.b1[i] = P[ob1 + i];
        L.b2[i] = P[ob2 + i];
        L.W3[i] = P[oW3 + i];
    }
    for (int i = threadIdx.x; i < kH * kH; i += blockDim.x) {
        L.W2[i] = (__bf16)P[oW2 + i];
    }
    if (threadIdx.x == 0) L.b3 = P[ob3];
    __syncthreads();
}

// Layer 1 for one row into the A-operand layout: h1[k] = relu(W1[k] . x + b1[k]) for
// k = 32 kb + 8 g + j.
__device__ __forceinline__ bf16x8 layer1_operand(const MlpLds& L, const float x[4], int kb, int g) {
    bf16x8 a;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = 32 * kb + 8 * g + j;
        float z = L.b1[k] + L.W1[4 * k] * x[0] + L.W1[4 * k + 1] * x[1] + L.W1[4 * k + 2] * x[2] + L.W1[4 * k + 3] * x[3];
        a[j] = (__bf16)fmaxf(z, 0.0f);
    }
    return a;
}

// B operand for the forward product: B[k][n] = W2[n][k], n = 16 nt + l % 16,
// k = 32 kb + 8 g + j (8 contiguous entries of row n of W2).
__device__ __forceinline__ bf16x8 w2_operand(const MlpLds& L, int nt, int kb, int lane) {
    const int n = 16 * nt + (lane & 15), g = lane >> 4;
    return *reinterpret_cast<const bf16x8*>(&L.W2[n * kH + 32 * kb + 8 * g]);
}

__device__ __forceinline__ float group16_sum(float v) {
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 8);
    return v;
}

// y = network(X) for n rows (X [n][4] FP32, y [n]).  Waves take 16-row tiles.
__global__ __launch_bounds__(kMlpBlock) void k_mlp_forward(int64_t n, const float4* __restrict__ X,
                                                           const float* __restrict__ P, float* __restrict__ y) {
    __shared__ MlpLds L;
    load_params(L, P);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, c = lane & 15;
    bf16x8 B[4][2];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) B[nt][kb] = w2_operand(L, nt, kb, lane);
    const int64_t n_tiles = (n + 15) / 16;
    for (int64_t t = (int64_t)blockIdx.x * 4 + wave; t < n_tiles; t += (int64_t)gridDim.x * 4) {
        const int64_t row = 16 * t + c;
        float x[4] = {0.f, 0.f, 0.f, 0.f};
        if (row < n) {
            const float4 v = X[row];
            x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
        }
        const bf16x8 a0 = layer1_operand(L, x, 0, g), a1 = layer1_operand(L, x, 1, g);
        float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
            acc = mfma(a0, B[nt][0], acc);
            acc = mfma(a1, B[nt][1], acc);
            const int nn = 16 * nt + c;
#pragma unroll
            for (int i = 0; i < 4; ++i) part[i] += fmaxf(acc[i] + L.b2[nn], 0.0f) * L.W3[nn];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float s = group16_sum(part[i]);
            const int64_t r = 16 * t + 4 * g + i;
            if (c == 0 && r < n) y[r] = s + L.b3;
        }
    }
}

// Minibatch source: explicit rows, or rows drawn from a recorded set by a counter-based
// hash of (seed, step, position).
struct BatchSrc {
    const float4* X;
    const float* T;
    int64_t n;            // rows in this minibatch
    int64_t n_all;        // rows in the recorded set (0 = explicit rows)
    uint64_t seed;
};

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ int64_t batch_row(const BatchSrc& s, int64_t i) {
    return s.n_all ? (int64_t)(mix64(s.seed ^ (uint64_t)i * 0xD1B54A32D192ED03ull) % (uint64_t)s.n_all) : i;
}

// Sum over each row of 16 lanes, in its last lane (DPP moves).
template <int kCtrl>
__device__ __forceinline__ float row_step(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}
__device__ __forceinline__ float row16_total(float v) {
    v = row_step<0x111>(v);   // row_shr:1
    v = row_step<0x112>(v);
    v = row_step<0x114>(v);
    return row_step<0x118>(v);
}

// Gradient of L = (1/N) sum (y - t)^2 over a minibatch; every workgroup writes the sum of
// its rows' gradients (4545 values) and of its squared errors to part[blockIdx].
// A workgroup takes tiles of 128 rows, wave w rows 32 w to 32 w + 31 in two halves of 16.
// The second layer is formed transposed, Z2^T = W2 H1^T (both operands as built for the
// plain product, swapped), so that lane (c, g) holds row c's units 16 nt + 4 g + i: the
// output and its error need two shuffles, and the rows' dz are, as they stand, the operand
// of dH1 = dZ2 W2 with the units of a K block in the order 32 kb + 4 g + i,
// 32 kb + 16 + 4 g + i, for which W2's columns are loaded into registers once.  dW2 = dZ2^T H1
// runs over the rows, which no lane holds together: dZ2 and H1 go transposed through LDS,
// shared by the workgroup, and wave w forms units 16 w to 16 w + 15 over all 128 rows, so
// that no sum across waves is left.  Bound by latency (one wave per SIMD; about 3.6 us per
// tile and 8 us of set-up and final sums): 65,536 rows 34.9 -> 18.5 us (32-row tiles per
// wave, all of dW2 in every wave and summed in LDS, 128 workgroups: 24.3 with 256 of them);
// 32,768 rows 14.9, 128 rows 12.1.  W2 staged in LDS first instead of read by every wave: 19.0.
constexpr int kTileRows = 128;
constexpr int kTileStride = kTileRows + 8;   // spreads the rows of the transposed tiles over the banks

__global__ __launch_bounds__(kMlpBlock) void k_mlp_grad(BatchSrc src, float inv_n, const float* __restrict__ P,
                                                        float* __restrict__ part, double* __restrict__ loss_part) {
    __shared__ float sW1[kH * kIn], sb1[kH], sb2[kH], sW3[kH];
    __shared__ alignas(16) __bf16 sZT[kH * kTileStride];   // [unit][row]
    __shared__ alignas(16) __bf16 sHT[kH * kTileStride];
    __shared__ float sX[4][32 * 4];
    __shared__ float sVec[4][7 * kH];
    __shared__ float sB3[4];
    __shared__ double sLoss[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, c = lane & 15;
    for (int i = threadIdx.x; i < kH * kIn; i += kMlpBlock) sW1[i] = P[oW1 + i];
    if (threadIdx.x < kH) {
        sb1[threadIdx.x] = P[ob1 + threadIdx.x];
        sb2[threadIdx.x] = P[ob2 + threadIdx.x];
        sW3[threadIdx.x] = P[oW3 + threadIdx.x];
    }
    const float b3 = P[ob3];
    // W2 rows for the forward product: row 16 nt + c, inputs 32 kb + 8 g + j; W2 columns for
    // the backward one: column 16 kt + c, units in the order above
    bf16x8 Wf[4][2], Wb[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                Wf[t][kb][j] = (__bf16)P[oW2 + (16 * t + c) * kH + 32 * kb + 8 * g + j];
                Wb[t][kb][j] = (__bf16)P[oW2 + (32 * kb + 16 * (j >> 2) + 4 * g + (j & 3)) * kH + 16 * t + c];
            }
    __syncthreads();

    floatx4 dW2[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) dW2[kt] = floatx4{0.f, 0.f, 0.f, 0.f};
    float dW1[4][4] = {}, db1[4] = {}, db2[4][4] = {}, dW3[4][4] = {};
    float db3 = 0.f;
    double loss = 0.0;

    const int64_t n_tiles = (src.n + kTileRows - 1) / kTileRows;
    for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        bf16x8 dz[2][2];   // [half][kb]
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int m = 32 * wave + 16 * h + c;   // the lane's row of the tile
            const int64_t i = t * kTileRows + m;
            float x[4] = {0.f, 0.f, 0.f, 0.f}, target = 0.f;
            if (i < src.n) {
                const int64_t r = batch_row(src, i);
                const float4 v = src.X[r];
                x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
                target = src.T[r];
            }
            if (g == 0) *reinterpret_cast<float4*>(&sX[wave][(16 * h + c) * 4]) = make_float4(x[0], x[1], x[2], x[3]);
            bf16x8 a[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = 32 * kb + 8 * g + j;
                    const float z = sb1[k] + sW1[4 * k] * x[0] + sW1[4 * k + 1] * x[1] + sW1[4 * k + 2] * x[2] +
                                    sW1[4 * k + 3] * x[3];
                    a[kb][j] = (__bf16)fmaxf(z, 0.0f);
                    sHT[k * kTileStride + m] = a[kb][j];
                }
            floatx4 z2[4];
            // the output in k_mlp_forward's order of sums (per unit mod 16, then pairwise), so that
            // the loss is the forward pass's own
            float part_y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma(Wf[nt][0], a[0], acc);
                acc = mfma(Wf[nt][1], a[1], acc);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = 16 * nt + 4 * g + q;
                    acc[q] += sb2[n];
                    part_y[q] += fmaxf(acc[q], 0.0f) * sW3[n];
                }
                z2[nt] = acc;
            }
            float y = (part_y[0] + part_y[1]) + (part_y[2] + part_y[3]);
            y += __shfl_xor(y, 16);
            y += __shfl_xor(y, 32);
            const float e = i < src.n ? y + b3 - target : 0.f;
            const float dy = 2.0f * inv_n * e;
            if (g == 0) {
                loss += (double)e * e;
                db3 += dy;
            }
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = 16 * nt + 4 * g + q;
                    const float z = z2[nt][q];
                    dW3[nt][q] += dy * fmaxf(z, 0.0f);
                    const float d = (z > 0.0f) ? dy * sW3[n] : 0.0f;
                    db2[nt][q] += d;
                    const __bf16 db = (__bf16)d;
                    dz[h][nt >> 1][4 * (nt & 1) + q] = db;
                    sZT[n * kTileStride + m] = db;
                }
        }
        __syncthreads();
        // ---- dW2[n][k] += sum over the tile's rows of dZ2[m][n] H1[m][k], n in 16 w .. 16 w + 15
#pragma unroll
        for (int s = 0; s < kTileRows / 32; ++s) {
            const int m0 = 32 * s + 8 * g;
            const bf16x8 za = *reinterpret_cast<const bf16x8*>(&sZT[(16 * wave + c) * kTileStride + m0]);
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                const bf16x8 hb = *reinterpret_cast<const bf16x8*>(&sHT[(16 * kt + c) * kTileStride + m0]);
                dW2[kt] = mfma(za, hb, dW2[kt]);
            }
        }
        // ---- dH1 = dZ2 W2 per half (rows 4 g + i, input 16 kt + c), then through the first ReLU
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                const int k = 16 * kt + c;
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma(dz[h][0], Wb[kt][0], acc);
                acc = mfma(dz[h][1], Wb[kt][1], acc);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 xr = *reinterpret_cast<const float4*>(&sX[wave][(16 * h + 4 * g + q) * 4]);
                    const float z1 = sb1[k] + sW1[4 * k] * xr.x + sW1[4 * k + 1] * xr.y + sW1[4 * k + 2] * xr.z +
                                     sW1[4 * k + 3] * xr.w;
                    const float dz1 = (z1 > 0.0f) ? acc[q] : 0.0f;
                    db1[kt] += dz1;
                    dW1[kt][0] += dz1 * xr.x;
                    dW1[kt][1] += dz1 * xr.y;
                    dW1[kt][2] += dz1 * xr.z;
                    dW1[kt][3] += dz1 * xr.w;
                }
            }
        __syncthreads();   // the tile has been read before the next one is written
    }

    // ---- part[blockIdx.x][0..4544]: dW2 as the waves hold it, the rest summed over lanes and waves
    float* out = part + (size_t)blockIdx.x * kNP;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int q = 0; q < 4; ++q) out[oW2 + (16 * wave + 4 * g + q) * kH + 16 * kt + c] = dW2[kt][q];
    float* vec = sVec[wave];   // dW1 [4 k + q], db1, db2, dW3
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
        const int k = 16 * kt + c;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v = dW1[kt][q];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (g == 0) vec[4 * k + q] = v;
        }
        float v = db1[kt];
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        if (g == 0) vec[4 * kH + k] = v;
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int n = 16 * nt + 4 * g + q;
            const float v2 = row16_total(db2[nt][q]), v3 = row16_total(dW3[nt][q]);
            if (c == 15) {
                vec[5 * kH + n] = v2;
                vec[6 * kH + n] = v3;
            }
        }
    for (int off = 8; off > 0; off >>= 1) {   // lanes of group 0 hold the rows' sums
        db3 += __shfl_xor(db3, off);
        loss += __shfl_xor(loss, off);
    }
    if (lane == 0) {
        sB3[wave] = db3;
        sLoss[wave] = loss;
    }
    __syncthreads();
    for (int v = threadIdx.x; v < 7 * kH; v += kMlpBlock) {
        const float a = (sVec[0][v] + sVec[1][v]) + (sVec[2][v] + sVec[3][v]);
        const int at = v < 5 * kH ? v : v < 6 * kH ? ob2 + v - 5 * kH : oW3 + v - 6 * kH;
        static_assert(oW1 == 0 && ob1 == 4 * kH, "W1 and b1 lead the parameters");
        out[at] = a;
    }
    if (threadIdx.x == 0) {
        out[ob3] = (sB3[0] + sB3[1]) + (sB3[2] + sB3[3]);
        loss_part[blockIdx.x] = (sLoss[0] + sLoss[1]) + (sLoss[2] + sLoss[3]);
    }
}

// grad[p] = sum over blocks (fixed order); optional Adam update of the FP32 masters.  A
// workgroup takes kRedParams parameters, kRedParts threads each summing every
// kRedParts-th partial (loads of 128 contiguous bytes, eight in flight), so that 143
// workgroups share what was a serial sum of all partials in 18: 31 -> 4.2 us for 65,536 rows.
// loss (optional): the mean squared error from the partial sums, by workgroup 0.
constexpr int kRedParams = 32, kRedParts = 8;

__global__ __launch_bounds__(256) void k_mlp_reduce_adam(const float* __restrict__ part, int n_blocks,
                                                         float* __restrict__ grad, float* __restrict__ P,
                                                         float* __restrict__ m, float* __restrict__ v, int adam,
                                                         float lr, float b1, float b2, float eps, float bc1, float bc2,
                                                         const double* __restrict__ loss_part, double inv_n,
                                                         double* __restrict__ loss) {
    static_assert(kRedParams * kRedParts == 256, "one thread per parameter and share");
    __shared__ float s_sum[kRedParts][kRedParams];
    __shared__ double s_loss[4];
    const int k = threadIdx.x % kRedParams, q = threadIdx.x / kRedParams;
    const int p = blockIdx.x * kRedParams + k;
    float a = 0.f;
    if (p < kNP) {
#pragma unroll 8
        for (int b = q; b < n_blocks; b += kRedParts) a += part[(size_t)b * kNP + p];
    }
    s_sum[q][k] = a;
    if (loss && blockIdx.x == 0) {
        double l = 0.0;
        for (int b = threadIdx.x; b < n_blocks; b += 256) l += loss_part[b];
        for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off);
        if ((threadIdx.x & 63) == 0) s_loss[threadIdx.x >> 6] = l;
    }
    __syncthreads();
    if (loss && blockIdx.x == 0 && threadIdx.x == 0) loss[0] = ((s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3])) * inv_n;
    if (q != 0 || p >= kNP) return;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kRedParts; ++w) s += s_sum[w][k];
    if (grad) grad[p] = s;
    if (adam) {
        const float mm = b1 * m[p] + (1.f - b1) * s;
        const float vv = b2 * v[p] + (1.f - b2) * s * s;
        m[p] = mm;
        v[p] = vv;
        P[p] -= lr * (mm / bc1) / (sqrtf(vv / bc2) + eps);
    }
}

// Per-edge features over the interior edges: e / s_e, (e - e_prev) / s_d,
// (e_prev - e_prev2) / s_d (differences in FP64, before the rounding), dG / s_g.
__global__ __launch_bounds__(256) void k_mlp_features(int64_t n_int, const int32_t* __restrict__ ie,
                                                      const double* __restrict__ e, const double* __restrict__ ep,
                                                      const double* __restrict__ ep2, const double* __restrict__ dg,
                                                      const double* __restrict__ scales, float4* __restrict__ X) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n_int) return;
    const int k = ie[j];
    const double se = 1.0 / scales[4], sd = 1.0 / scales[0], sg = 1.0 / scales[1];
    const double en = e[k], e1 = ep[k];
    X[j] = make_float4((float)(en * se), (float)((en - e1) * sd), (float)((e1 - ep2[k]) * sd), (float)(dg[k] * sg));
}

// The scales of the inputs over interior edges (each 1 where zero): s_d = RMS of
// e^n - e^{n-1} into scales[0], s_g = RMS of dG into scales[1], s_e = RMS of e^n into
// scales[4]; per-workgroup sums of squares (grid-stride), then one workgroup adds them in
// a fixed order.
constexpr int kRmsBlocks = 256;

__global__ __launch_bounds__(256) void k_mlp_rms_part(int64_t n_int, const int32_t* __restrict__ ie,
                                                      const double* __restrict__ e, const double* __restrict__ ep,
                                                      const double* __restrict__ dg, double* __restrict__ part) {
    __shared__ double s[3][4];
    double a = 0.0, b = 0.0, c = 0.0;
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n_int; j += (int64_t)gridDim.x * 256) {
        const int k = ie[j];
        const double en = e[k], d = en - ep[k], g = dg[k];
        a += en * en;
        b += d * d;
        c += g * g;
    }
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off);
        b += __shfl_xor(b, off);
        c += __shfl_xor(c, off);
    }
    if ((threadIdx.x & 63) == 0) {
        s[0][threadIdx.x >> 6] = a;
        s[1][threadIdx.x >> 6] = b;
        s[2][threadIdx.x >> 6] = c;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int q = threadIdx.x;
        part[q * kRmsBlocks + blockIdx.x] = (s[q][0] + s[q][1]) + (s[q][2] + s[q][3]);
    }
}

__global__ __launch_bounds__(256) void k_mlp_rms_fin(int64_t n_int, int nb, const double* __restrict__ part,
                                                     double* __restrict__ scales) {
    __shared__ double s[3][4];
    double v[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) v[q] = threadIdx.x < nb ? part[q * kRmsBlocks + threadIdx.x] : 0.0;
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] += __shfl_xor(v[q], off);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int q = 0; q < 3; ++q) s[q][threadIdx.x >> 6] = v[q];
    __syncthreads();
    if (threadIdx.x == 0) {
        double r[3];
        for (int q = 0; q < 3; ++q) {
            const double sum = (s[q][0] + s[q][1]) + (s[q][2] + s[q][3]);
            r[q] = n_int ? sqrt(sum / (double)n_int) : 0.0;
            if (!(r[q] > 0.0)) r[q] = 1.0;
        }
        scales[4] = r[0];
        scales[0] = r[1];
        scales[1] = r[2];
    }
}

// Rows r0, r0 + stride, ... (n of them) of X [rows][4] into dst: the subsample of edges a
// snapshot records.
__global__ __launch_bounds__(256) void k_mlp_pick(const float4* __restrict__ X, int64_t r0, int64_t stride, int64_t n,
                                                  float4* __restrict__ dst) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < n) dst[j] = X[r0 + j * stride];
}

// Predicted increment as an edge vector: d[ie] = s_d y (d is zero elsewhere).
__global__ __launch_bounds__(256) void k_mlp_direction(int64_t n_int, const int32_t* __restrict__ ie,
                                                       const float* __restrict__ y, const double* __restrict__ scales,
                                                       double* __restrict__ d) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n_int) return;
    d[ie[j]] = scales[0] * (double)y[j];
}

// Training target, first pass: the increments e^{n+1} - e^n on interior edges r0,
// r0 + stride, ... (n rows) into d (FP64) and per-workgroup sums of their squares.
__global__ __launch_bounds__(256) void k_mlp_target(int64_t n, int64_t r0, int64_t stride,
                                                    const int32_t* __restrict__ ie, const double* __restrict__ e_new,
                                                    const double* __restrict__ e, double* __restrict__ d,
                                                    double* __restrict__ part) {
    __shared__ double s[4];
    double a = 0.0;
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
        const int k = ie[r0 + j * stride];
        const double v = e_new[k] - e[k];
        d[j] = v;
        a += v * v;
    }
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (s[0] + s[1]) + (s[2] + s[3]);
}

// Second pass: t = d / s_d, and (workgroup 0) the RMS of t into scales[3], by which the host
// leaves out steps where the history is near zero (a neutral start) and the increment
// dwarfs it.
__global__ __launch_bounds__(256) void k_mlp_target_scale(int64_t n, int nb, const double* __restrict__ part,
                                                          const double* __restrict__ d, double* __restrict__ scales,
                                                          float* __restrict__ t) {
    const double inv = 1.0 / scales[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        double a = 0.0;
        for (int b = 0; b < nb; ++b) a += part[b];
        scales[3] = n ? sqrt(a / (double)n) * inv : 0.0;
    }
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256)
        t[j] = (float)(d[j] * inv);
}

}  // namespace

// ------------------------------------------------------------------------- launchers
// One workgroup per tile of 128 rows up to one per CU (every workgroup writes and the
// reduction reads 18 KB of partial sums).
constexpr int kMaxGradGrid = 256;
int mlp_grad_blocks(int64_t n) {
    const int64_t tiles = (n + kTileRows - 1) / kTileRows;
    return (int)std::min<int64_t>(std::max<int64_t>(tiles, 1), kMaxGradGrid);
}

void mlp_launch_rms(hipStream_t s, int64_t n_int, const int32_t* ie, const double* e, const double* ep,
                    const double* dg, double* part, double* scales) {
    const int nb = (int)std::max<int64_t>(1, std::min<int64_t>(kRmsBlocks, (n_int + 1023) / 1024));
    hipLaunchKernelGGL(k_mlp_rms_part, dim3(nb), dim3(256), 0, s, n_int, ie, e, ep, dg, part);
    hipLaunchKernelGGL(k_mlp_rms_fin, dim3(1), dim3(256), 0, s, n_int, nb, part, scales);
}

void mlp_launch_features(hipStream_t s, int64_t n_int, const int32_t* ie, const double* e, const double* ep,
                         const double* ep2, const double* dg, const double* scales, float* X) {
    if (n_int <= 0) return;
    hipLaunchKernelGGL(k_mlp_features, dim3(grid_1d(n_int, 256)), dim3(256), 0, s, n_int, ie, e, ep, ep2, dg, scales,
                       (float4*)X);
}

void mlp_launch_forward(hipStream_t s, int64_t n, const float* X, const float* P, float* y) {
    if (n <= 0) return;
    const int64_t tiles = (n + 15) / 16;
    int64_t blocks = (tiles + 3) / 4;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)blocks), dim3(kMlpBlock), 0, s, n, (const float4*)X, P, y);
}

void mlp_launch_direction(hipStream_t s, int64_t n_int, const int32_t* ie, const float* y, const double* scales,
                          double* d) {
    if (n_int <= 0) return;
    hipLaunchKernelGGL(k_mlp_direction, dim3(grid_1d(n_int, 256)), dim3(256), 0, s, n_int, ie, y, scales, d);
}

void mlp_launch_target(hipStream_t s, int64_t n, int64_t r0, int64_t stride, const int32_t* ie, const double* e_new,
                       const double* e, double* work, double* part, double* scales, float* t) {
    if (n <= 0) return;
    const int nb = (int)std::max<int64_t>(1, std::min<int64_t>(kRmsBlocks, (n + 1023) / 1024));
    hipLaunchKernelGGL(k_mlp_target, dim3(nb), dim3(256), 0, s, n, r0, stride, ie, e_new, e, work, part);
    hipLaunchKernelGGL(k_mlp_target_scale, dim3(nb), dim3(256), 0, s, n, nb, part, work, scales, t);
}

void mlp_launch_pick(hipStream_t s, const float* X, int64_t r0, int64_t stride, int64_t n, float* dst) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_mlp_pick, dim3(grid_1d(n, 256)), dim3(256), 0, s, (const float4*)X, r0, stride, n,
                       (float4*)dst);
}

void mlp_launch_grad(hipStream_t s, const float* X, const float* T, int64_t n, int64_t n_all, uint64_t seed,
                     const float* P, float* part, double* loss_part, int blocks) {
    BatchSrc src{(const float4*)X, T, n, n_all, seed};
    hipLaunchKernelGGL(k_mlp_grad, dim3(blocks), dim3(kMlpBlock), 0, s, src, 1.0f / (float)n, P, part, loss_part);
}

void mlp_launch_reduce_adam(hipStream_t s, const float* part, int blocks, float* grad, float* P, float* m, float* v,
                            int adam, float lr, float b1, float b2, float eps, float bc1, float bc2,
                            const double* loss_part, double inv_n, double* loss) {
    hipLaunchKernelGGL(k_mlp_reduce_adam, dim3((kNP + kRedParams - 1) / kRedParams), dim3(256), 0, s, part, blocks, grad, P,
                       m, v, adam, lr, b1, b2, eps, bc1, bc2, loss_part, inv_n, loss);
}

}  // namespace fepic
