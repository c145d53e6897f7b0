// Training and inference kernels of the learned Newton initial guess
// (include/fr_dvm_mlp.h), FP32 on gfx950.
//
// The dense layers are small GEMMs (batch x 64 x 64) run on the matrix cores
// with v_mfma_f32_16x16x4_f32.  Up to 64 hidden neurons all layers of a row
// block run in one kernel, forward, backward and weight gradients; wider
// networks run layer by layer (one wave per 16x16 output tile, K stepped by
// 4; bias/activation, loss and column sums as plain elementwise kernels).
// Every reduction has a fixed order, so training is bitwise reproducible.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <mutex>

#include "../../include/fr_dvm_mlp.h"
#include "frdvm_common.h"

namespace frdvm {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// C[M][N] = sum_k A(m,k) B(k,n);  A(m,k) = tA ? A[k lda + m] : A[m lda + k],
// B(k,n) = tB ? B[n ldb + k] : B[k ldb + n].  Operand layout of the 16x16x4
// FP32 MFMA: lane l supplies A[l%16][l/16] and B[l/16][l%16] and receives
// D[4 (l/16) + i][l%16], i = 0..3.
__global__ __launch_bounds__(256) void k_gemm(int M, int N, int K, const float *__restrict__ A, int lda, int tA,
                                              const float *__restrict__ B, int ldb, int tB, float *__restrict__ C,
                                              int ldc) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int tilesN = (N + 15) / 16;
    const int tile = blockIdx.x * 4 + wave;
    const int tm = tile / tilesN, tn = tile % tilesN;
    if (tm * 16 >= M) return;  // whole wave leaves together
    const int r16 = lane & 15, q = lane >> 4;
    const int m = tm * 16 + r16, n = tn * 16 + r16;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += 4) {
        const int k = k0 + q;
        float a = 0.f, b = 0.f;
        if (m < M && k < K) a = tA ? A[(int64_t)k * lda + m] : A[(int64_t)m * lda + k];
        if (n < N && k < K) b = tB ? B[(int64_t)n * ldb + k] : B[(int64_t)k * ldb + n];
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int mm = tm * 16 + 4 * q + i, nn = tn * 16 + r16;
        if (mm < M && nn < N) C[(int64_t)mm * ldc + nn] = acc[i];
    }
}

__device__ __forceinline__ float silu(float x) { return x / (1.f + __expf(-x)); }
__device__ __forceinline__ float dsilu(float x) {
    float s = 1.f / (1.f + __expf(-x));
    return s * (1.f + x * (1.f - s));
}

// Z += bias (per column); A = silu(Z) when act, else nothing.
__global__ void k_bias_act(int64_t M, int N, float *Z, const float *bias, float *A, int act) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M * N) return;
    float z = Z[i] + bias[i % N];
    Z[i] = z;
    if (act) A[i] = silu(z);
}

// delta = (Y - T)/B in place of Y; per-block partial sums of |Y - T|^2 / (2B).
__global__ __launch_bounds__(256) void k_loss_delta(int64_t B, float *Y, const float *T, float *partial) {
    __shared__ float red[256];
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float l = 0.f;
    if (i < B * 5) {
        float r = Y[i] - T[i];
        l = 0.5f * r * r / (float)B;
        Y[i] = r / (float)B;
    }
    red[threadIdx.x] = l;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void k_sum(int n, const float *partial, float *out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        float s = 0.f;
        for (int i = 0; i < n; ++i) s += partial[i];
        out[0] = s;
    }
}

__global__ void k_dsilu_mul(int64_t n, float *D, const float *Z) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) D[i] *= dsilu(Z[i]);
}

// out[n] = sum over rows of D[m][n] (sequential per column: fixed order).
__global__ void k_colsum(int64_t M, int N, const float *D, float *out) {
    int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    float s = 0.f;
    for (int64_t m = 0; m < M; ++m) s += D[m * N + n];
    out[n] = s;
}

__global__ void k_adam(int64_t n, float *w, const float *g, float *m, float *v, float c1, float c2, float lr) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float mi = 0.9f * m[i] + 0.1f * g[i];
    float vi = 0.999f * v[i] + 0.001f * g[i] * g[i];
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
}

__global__ void k_affine(int64_t B, const float *Y, const float *scale, const float *offset, float *out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < B * 5) out[i] = Y[i] * scale[i % 5] + offset[i % 5];
}

struct Layout {
    size_t W[4], b[4], scale, offset, total;
    int in[4], out[4];
};

Layout layout(int H) {
    Layout L;
    int ins[4] = {FR_MLP_INPUTS, H, H, H}, outs[4] = {H, H, H, 5};
    size_t o = 0;
    for (int l = 0; l < 4; ++l) {
        L.in[l] = ins[l];
        L.out[l] = outs[l];
        L.W[l] = o;
        o += (size_t)outs[l] * ins[l];
        L.b[l] = o;
        o += outs[l];
    }
    L.scale = o;
    L.offset = o + 5;
    L.total = o + 10;
    return L;
}

struct Work {
    float *Z[3], *A[3], *Y, *Da, *Db, *partial;
};

Work carve(float *work, int H, int64_t B) {
    Work w;
    size_t bh = (size_t)B * H;
    for (int l = 0; l < 3; ++l) {
        w.Z[l] = work + (2 * l) * bh;
        w.A[l] = work + (2 * l + 1) * bh;
    }
    w.Y = work + 6 * bh;
    w.Da = w.Y + (size_t)B * 5;
    w.Db = w.Da + bh;
    w.partial = w.Db + bh;
    return w;
}

void gemm(hipStream_t s, int M, int N, int K, const float *A, int lda, int tA, const float *B, int ldb, int tB,
          float *C, int ldc) {
    int tiles = ((M + 15) / 16) * ((N + 15) / 16);
    hipLaunchKernelGGL(k_gemm, dim3((tiles + 3) / 4), dim3(256), 0, s, M, N, K, A, lda, tA, B, ldb, tB, C, ldc);
}

unsigned blocks(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// ---- one-kernel network passes for hidden widths up to 64 ----------------
//
// What bounds the network at training sizes is latency: a few thousand rows
// of 64-wide layers are 0.2 GFLOP, far below a launch's worth of matrix-core
// time, so a kernel per layer and per bias, activation, loss, column sum and
// weight-gradient product pays for launches and for reductions over the
// batch that leave the chip idle.  Here a workgroup of HT = ceil(H / 16)
// waves takes 16 rows of the batch through every layer: wave w owns the
// hidden neurons 16 w .. 16 w + 15, holds its weights as MFMA operands in
// registers for all its row blocks, and passes activations to the other
// waves through LDS.  Training adds the loss, the backward pass and the
// weight gradients in the same kernel (accumulated over the workgroup's row
// blocks in MFMA accumulators), one partial gradient per workgroup, and
// k_mlp_reduce adds the partials in a fixed order (bitwise reproducible).
// Batch 4096, H = 64, gradient and Adam step: 3782 us layer by layer (the
// column sums walked the batch in one wave per layer, the weight gradients in
// 16 tiles), 24 us so; a prediction of 65,536 rows 240 -> 55 us.
//
// MFMA operand layout (16x16x4 FP32): lane (r = l % 16, q = l / 16) supplies
// A[r][kk] and B[kk][r], kk = q, and receives D[4 q + i][r].  The kk of the
// j-th MFMA of a group of 16 k is 4 q + j, so that a lane reads its A values
// as one float4; and a tile in D layout (rows m = 4 q + i, i = j) is directly
// an operand of a product that sums over rows m, as the weight gradients do.
template <int HT>
struct MlpTile {
    static constexpr int HP = 16 * HT;      // padded width
    static constexpr int S = HP + 4;        // LDS row stride: 16-byte aligned rows, distinct banks
    static constexpr int SX = 20;           // the same for 16 inputs / 16 outputs
};

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Rows of the weight matrix W[out][in] as the B operand of a forward product:
// element [t][j] = W[n][16 t + 4 q + j], zero outside.
template <int KT>
__device__ __forceinline__ void load_fwd(const float *W, int out, int in, int n, int q, float (&b)[KT][4]) {
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 16 * t + 4 * q + j;
            b[t][j] = n < out && k < in ? W[n * in + k] : 0.f;
        }
}
// Columns of W as the B operand of a backward product: [t][j] = W[16 t + 4 q + j][c].
template <int KT>
__device__ __forceinline__ void load_bwd(const float *W, int out, int in, int c, int q, float (&b)[KT][4]) {
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = 16 * t + 4 * q + j;
            b[t][j] = n < out && c < in ? W[n * in + c] : 0.f;
        }
}
// 16 x 16 tile of A[16][16 KT] (LDS rows of stride ld) times the operand b.
template <int KT>
__device__ __forceinline__ floatx4 tile_product(const float *A, int ld, int r, int q, const float (&b)[KT][4]) {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        const floatx4 a = *reinterpret_cast<const floatx4 *>(A + r * ld + 16 * t + 4 * q);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = mfma4(a[j], b[t][j], acc);
    }
    return acc;
}

// GRAD: the gradient pass (partial gradient rows of `out`, or the gradient
// itself when the grid is one workgroup); else the prediction dz in `out`,
// times T[row] if T is given.
template <int HT, bool GRAD>
__global__ __launch_bounds__(64 * HT) void k_mlp_rows(const float *__restrict__ w, const float *__restrict__ X,
                                                      const float *__restrict__ T, int64_t B, int H, Layout L,
                                                      float *__restrict__ out, float *__restrict__ loss_out,
                                                      int64_t row_floats) {
    using G = MlpTile<HT>;
    constexpr int S = G::S, SX = G::SX;
    __shared__ __attribute__((aligned(16))) float sX[16 * SX];
    __shared__ __attribute__((aligned(16))) float sA[GRAD ? 3 : 2][16 * S];
    __shared__ __attribute__((aligned(16))) float sD[GRAD ? 2 : 1][GRAD ? 16 * S : 4];
    __shared__ __attribute__((aligned(16))) float sY[GRAD ? HT : 1][GRAD ? 16 * SX : 4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r = lane & 15, q = lane >> 4, n = 16 * wv + r;  // n: the lane's hidden neuron
    // operands of this wave, for all its row blocks
    float f0[1][4], f1[HT][4], f2[HT][4], f3[HT][4], bias[3], b3;
    load_fwd<1>(w + L.W[0], H, FR_MLP_INPUTS, n, q, f0);
    load_fwd<HT>(w + L.W[1], H, H, n, q, f1);
    load_fwd<HT>(w + L.W[2], H, H, n, q, f2);
    load_fwd<HT>(w + L.W[3], 5, H, r, q, f3);
#pragma unroll
    for (int l = 0; l < 3; ++l) bias[l] = n < H ? w[L.b[l] + n] : 0.f;
    b3 = r < 5 ? w[L.b[3] + r] : 0.f;
    float g1[GRAD ? HT : 1][4], g2[GRAD ? HT : 1][4], g3[1][4];
    floatx4 dW0 = {0, 0, 0, 0}, dW1[HT], dW2[HT], dW3 = {0, 0, 0, 0};
    float db[3] = {0.f, 0.f, 0.f}, db3 = 0.f, loss = 0.f;
    if constexpr (GRAD) {
        load_bwd<HT>(w + L.W[1], H, H, n, q, g1);
        load_bwd<HT>(w + L.W[2], H, H, n, q, g2);
        load_bwd<1>(w + L.W[3], 5, H, n, q, g3);
#pragma unroll
        for (int t = 0; t < HT; ++t) dW1[t] = dW2[t] = floatx4{0, 0, 0, 0};
    }
    float sc = 0.f, of = 0.f;
    if (!GRAD && r < 5) {
        sc = w[L.scale + r];
        of = w[L.offset + r];
    }
    const float fB = (float)B;
    const int64_t nblk = (B + 15) / 16;
    for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        const int64_t m0 = blk * 16;
        for (int i = threadIdx.x; i < 256; i += 64 * HT) {
            const int m = i >> 4, k = i & 15;
            sX[m * SX + k] = m0 + m < B && k < FR_MLP_INPUTS ? X[(m0 + m) * FR_MLP_INPUTS + k] : 0.f;
        }
        // the targets of the rows this lane holds in D layout
        float tgt[4] = {0.f, 0.f, 0.f, 0.f};
        if (GRAD && r < 5) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (m0 + 4 * q + i < B) tgt[i] = T[(m0 + 4 * q + i) * 5 + r];
        }
        __syncthreads();
        floatx4 a[3], ds[3];  // activations and SiLU derivatives of the wave's tile
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const floatx4 z = l == 0 ? tile_product<1>(sX, SX, r, q, f0)
                                     : (l == 1 ? tile_product<HT>(sA[0], S, r, q, f1) : tile_product<HT>(sA[1], S, r, q, f2));
            float *dst = sA[GRAD ? l : (l & 1)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                // (a neuron past the width stays 0 also where a real one is
                // infinite: 0 x inf would make the row NaN)
                const float x = z[i] + bias[l];
                a[l][i] = n < H ? silu(x) : 0.f;
                if (GRAD) ds[l][i] = dsilu(x);
                dst[(4 * q + i) * S + n] = a[l][i];
            }
            __syncthreads();
        }
        if constexpr (!GRAD) {
            // (written by wave 0; the barriers of the next block order its LDS reads before their rewrite)
            if (wv == 0) {
                const floatx4 y = tile_product<HT>(sA[0], S, r, q, f3);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (r < 5 && m0 + 4 * q + i < B) {
                        const float v = (y[i] + b3) * sc + of;
                        out[(m0 + 4 * q + i) * 5 + r] = T ? v * T[m0 + 4 * q + i] : v;
                    }
            }
            continue;
        }
        if constexpr (GRAD) {
            // output layer in every wave (its delta is an operand of each)
            const floatx4 y = tile_product<HT>(sA[2], S, r, q, f3);
            floatx4 d3 = {0, 0, 0, 0};
            float *sy = sY[wv];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (r < 5 && m0 + 4 * q + i < B) {
                    const float e = y[i] + b3 - tgt[i];
                    loss += 0.5f * e * e / fB;
                    d3[i] = e / fB;
                }
                db3 += d3[i];
                sy[(4 * q + i) * SX + r] = d3[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            floatx4 d = tile_product<1>(sy, SX, r, q, g3);
#pragma unroll
            for (int j = 0; j < 4; ++j) dW3 = mfma4(d3[j], a[2][j], dW3);  // [output][own tile]
#pragma unroll
            for (int l = 2; l >= 0; --l) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    d[i] = n < H ? d[i] * ds[l][i] : 0.f;
                    db[l] += d[i];
                    if (l > 0) sD[l - 1][(4 * q + i) * S + n] = d[i];
                }
                if (l == 0) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) dW0 = mfma4(d[j], sX[(4 * q + j) * SX + r], dW0);
                    break;
                }
                // weight gradient of the wave's rows against every tile of the layer's input
#pragma unroll
                for (int t = 0; t < HT; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        floatx4 &acc = l == 2 ? dW2[t] : dW1[t];
                        acc = mfma4(d[j], sA[l - 1][(4 * q + j) * S + 16 * t + r], acc);
                    }
                __syncthreads();
                d = l == 2 ? tile_product<HT>(sD[1], S, r, q, g2) : tile_product<HT>(sD[0], S, r, q, g1);
            }
            __syncthreads();  // the tiles are rewritten by the next block
        }
    }
    if constexpr (GRAD) {
        float *o = out + blockIdx.x * row_floats;
        auto over_q = [&](float v) {  // sum over the four row groups of a column
            v += __shfl_xor(v, 16);
            return v + __shfl_xor(v, 32);
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = 16 * wv + 4 * q + i;  // neuron (row of the weight matrix)
            if (m < H) {
                if (r < FR_MLP_INPUTS) o[L.W[0] + m * FR_MLP_INPUTS + r] = dW0[i];
#pragma unroll
                for (int t = 0; t < HT; ++t)
                    if (16 * t + r < H) {
                        o[L.W[1] + m * H + 16 * t + r] = dW1[t][i];
                        o[L.W[2] + m * H + 16 * t + r] = dW2[t][i];
                    }
            }
            if (4 * q + i < 5 && n < H) o[L.W[3] + (4 * q + i) * H + n] = dW3[i];
        }
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const float v = over_q(db[l]);
            if (q == 0 && n < H) o[L.b[l] + n] = v;
        }
        if (wv == 0) {
            const float v = over_q(db3);
            if (q == 0 && r < 5) o[L.b[3] + r] = v;
            float s = over_q(loss);
#pragma unroll
            for (int x = 8; x >= 1; x >>= 1) s += __shfl_xor(s, x);
            if (lane == 0) *(gridDim.x == 1 ? loss_out : o + L.scale) = s;
        }
        // the output affine has no gradient
        if (gridDim.x == 1 && threadIdx.x < 10) o[L.scale + threadIdx.x] = 0.f;
    }
}

// Sum of the workgroups' partial gradients [nwg][np + 1] (the last entry the
// loss) in workgroup order per slice, the kSlices slices added in order:
// 16 consecutive parameters by 16 slices per block, so that a block has many
// loads in flight.  The 10 affine entries of grad are zero.
constexpr int kSlices = 16;
__global__ __launch_bounds__(256) void k_mlp_reduce(int nwg, int np, const float *__restrict__ part,
                                                    float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float red[kSlices][17];
    const int c = threadIdx.x & 15, sl = threadIdx.x >> 4;
    const int p = blockIdx.x * 16 + c;
    float s = 0.f;
    if (p <= np) {
#pragma unroll 4
        for (int g = sl; g < nwg; g += kSlices) s += part[(int64_t)g * (np + 1) + p];
    }
    red[sl][c] = s;
    __syncthreads();
    if (sl == 0 && p <= np) {
        float t = red[0][c];
#pragma unroll
        for (int g = 1; g < kSlices; ++g) t += red[g][c];
        if (p < np) grad[p] = t;
        else loss[0] = t;
    }
    if (blockIdx.x == 0 && threadIdx.x < 10) grad[np + threadIdx.x] = 0.f;
}

// Widest network of the one-kernel passes: four 16-wide tiles of neurons hold
// every layer's weights of a wave in registers.  Wider ones run layer by layer.
constexpr int kRowsMaxH = 64;

template <bool GRAD>
void launch_rows(hipStream_t s, int H, unsigned nwg, const float *w, const float *X, const float *T, int64_t B,
                 float *out, float *loss, int64_t row_floats) {
    const Layout L = layout(H);
    switch ((H + 15) / 16) {
        case 1: hipLaunchKernelGGL((k_mlp_rows<1, GRAD>), dim3(nwg), dim3(64), 0, s, w, X, T, B, H, L, out, loss, row_floats); break;
        case 2: hipLaunchKernelGGL((k_mlp_rows<2, GRAD>), dim3(nwg), dim3(128), 0, s, w, X, T, B, H, L, out, loss, row_floats); break;
        case 3: hipLaunchKernelGGL((k_mlp_rows<3, GRAD>), dim3(nwg), dim3(192), 0, s, w, X, T, B, H, L, out, loss, row_floats); break;
        default: hipLaunchKernelGGL((k_mlp_rows<4, GRAD>), dim3(nwg), dim3(256), 0, s, w, X, T, B, H, L, out, loss, row_floats);
    }
}

// Prediction of a batch: up to four workgroups per CU, each looping over its
// row blocks with the weights in registers.
void forward_rows(hipStream_t s, int H, const float *w, const float *X, int64_t B, float *dz,
                  const float *env = nullptr) {
    const int64_t nblk = (B + 15) / 16;
    launch_rows<false>(s, H, (unsigned)(nblk < 1024 ? nblk : 1024), w, X, env, B, dz, nullptr, 0);
}

// Forward pass into the workspace; Y holds the normalised output.
void forward(hipStream_t s, int H, const float *w, const float *X, int64_t B, const Work &wk) {
    Layout L = layout(H);
    const float *a = X;
    for (int l = 0; l < 3; ++l) {
        gemm(s, (int)B, H, L.in[l], a, L.in[l], 0, w + L.W[l], L.in[l], 1, wk.Z[l], H);
        hipLaunchKernelGGL(k_bias_act, dim3(blocks(B * H)), dim3(256), 0, s, B, H, wk.Z[l], w + L.b[l], wk.A[l], 1);
        a = wk.A[l];
    }
    gemm(s, (int)B, 5, H, a, H, 0, w + L.W[3], H, 1, wk.Y, 5);
    hipLaunchKernelGGL(k_bias_act, dim3(blocks(B * 5)), dim3(256), 0, s, B, 5, wk.Y, w + L.b[3], (float *)nullptr, 0);
}

// Scratch of fr_mlp_forward_noalloc: two [B][H] activation buffers used in
// turn (each layer's GEMM writes one from the other, bias and SiLU in place)
// and the [B][5] output.  In host code `scratch` names a host-side stand-in;
// kernels receive the device address from hipGetSymbolAddress, kept per GPU.
static __device__ __align__(256) float scratch[FR_MLP_NOALLOC_FLOATS];

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
float *scratch_dev[kMaxDevices] = {};

// Device address of the current GPU's scratch, looked up once per GPU with
// that GPU current.
int scratch_ptr(float **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return FR_DVM_EHIP;
    if (dev < 0 || dev >= kMaxDevices) return FR_DVM_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_dev[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return FR_DVM_EHIP;
        scratch_dev[dev] = static_cast<float *>(ptr);
    }
    *out = scratch_dev[dev];
    return FR_DVM_OK;
}

int hip_ok(const char *what) {
    (void)what;
    return hipGetLastError() == hipSuccess ? FR_DVM_OK : FR_DVM_EHIP;
}

}  // namespace

int mlp_forward_scaled(int H, const float *w, const float *X, int64_t B, const float *env, float *dz, hipStream_t s) {
    if (H < 1 || H > kRowsMaxH) return FR_DVM_EUNSUPPORTED;
    forward_rows(s, H, w, X, B, dz, env);
    return hip_ok("mlp forward");
}

}  // namespace frdvm

using namespace frdvm;

extern "C" size_t fr_mlp_param_count(int H) { return H > 0 ? layout(H).total : 0; }

extern "C" size_t fr_mlp_workspace_floats(int H, int64_t B) {
    return (size_t)8 * B * H + (size_t)5 * B + ((size_t)B * 5 + 255) / 256 + 16;
}

extern "C" int fr_mlp_forward(int H, const float *w, const float *X, int64_t B, float *dz, float *work, void *stream) {
    if (H < 1 || H > 1024 || B < 0 || !w || !work || (B > 0 && (!X || !dz))) return FR_DVM_EINVAL;
    if (B == 0) return FR_DVM_OK;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (H <= kRowsMaxH) {
        forward_rows(s, H, w, X, B, dz);
        return hip_ok("mlp forward");
    }
    Work wk = carve(work, H, B);
    forward(s, H, w, X, B, wk);
    Layout L = layout(H);
    hipLaunchKernelGGL(k_affine, dim3(blocks(B * 5)), dim3(256), 0, s, B, wk.Y, w + L.scale, w + L.offset, dz);
    return hip_ok("mlp forward");
}

extern "C" int fr_mlp_forward_noalloc(int H, const float *w, const float *X, int64_t B, float *dz, void *stream) {
    if (H < 1 || H > 1024 || B < 0 || !w || (B > 0 && (!X || !dz))) return FR_DVM_EINVAL;
    if (B == 0) return FR_DVM_OK;
    if ((size_t)B > FR_MLP_NOALLOC_FLOATS / (size_t)(2 * H + 5)) return FR_DVM_ESCRATCH;
    if (H <= kRowsMaxH) {
        forward_rows(reinterpret_cast<hipStream_t>(stream), H, w, X, B, dz);
        return hip_ok("mlp forward (no allocation)");
    }
    float *base = nullptr;
    int rc = scratch_ptr(&base);
    if (rc) return rc;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    Layout L = layout(H);
    float *act[2] = {base, base + (size_t)B * H};
    float *Y = base + (size_t)2 * B * H;
    const float *a = X;
    for (int l = 0; l < 3; ++l) {
        float *z = act[l & 1];
        gemm(s, (int)B, H, L.in[l], a, L.in[l], 0, w + L.W[l], L.in[l], 1, z, H);
        hipLaunchKernelGGL(k_bias_act, dim3(blocks(B * H)), dim3(256), 0, s, B, H, z, w + L.b[l], z, 1);
        a = z;
    }
    gemm(s, (int)B, 5, H, a, H, 0, w + L.W[3], H, 1, Y, 5);
    hipLaunchKernelGGL(k_bias_act, dim3(blocks(B * 5)), dim3(256), 0, s, B, 5, Y, w + L.b[3], (float *)nullptr, 0);
    hipLaunchKernelGGL(k_affine, dim3(blocks(B * 5)), dim3(256), 0, s, B, Y, w + L.scale, w + L.offset, dz);
    return hip_ok("mlp forward (no allocation)");
}

extern "C" int fr_mlp_grad(int H, const float *w, const float *X, const float *T, int64_t B, float *grad, float *loss,
                           float *work, void *stream) {
    if (H < 1 || H > 1024 || B < 1 || !w || !X || !T || !grad || !loss || !work) return FR_DVM_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    Layout L = layout(H);
    if (H <= kRowsMaxH) {
        // one partial gradient (and loss) per workgroup, as many workgroups
        // as row blocks, CUs and the workspace allow; with one, the kernel
        // writes the gradient itself
        const int64_t nblk = (B + 15) / 16, row = (int64_t)L.scale + 1;
        int64_t most = (int64_t)fr_mlp_workspace_floats(H, B) / row;
        if (most > 256) most = 256;
        if (most < 1) most = 1;
        const int64_t per = (nblk + most - 1) / most, nwg = (nblk + per - 1) / per;
        launch_rows<true>(s, H, (unsigned)nwg, w, X, T, B, nwg == 1 ? grad : work, loss, row);
        if (nwg > 1)
            hipLaunchKernelGGL(k_mlp_reduce, dim3((unsigned)((row + 15) / 16)), dim3(256), 0, s, (int)nwg,
                               (int)L.scale, work, grad, loss);
        return hip_ok("mlp grad");
    }
    Work wk = carve(work, H, B);
    forward(s, H, w, X, B, wk);
    const unsigned nb = blocks(B * 5);
    hipLaunchKernelGGL(k_loss_delta, dim3(nb), dim3(256), 0, s, B, wk.Y, T, wk.partial);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(64), 0, s, (int)nb, wk.partial, loss);
    // output layer: delta in Y [B][5]
    const float *delta = wk.Y;
    int dn = 5;
    float *bufs[2] = {wk.Da, wk.Db};
    for (int l = 3; l >= 0; --l) {
        const float *ain = l == 0 ? X : wk.A[l - 1];
        const int nin = L.in[l];
        // dW_l = delta^T a_in  (out x in), db_l = column sums of delta
        gemm(s, dn, nin, (int)B, delta, dn, 1, ain, nin, 0, grad + L.W[l], nin);
        hipLaunchKernelGGL(k_colsum, dim3(blocks(dn, 64)), dim3(64), 0, s, B, dn, delta, grad + L.b[l]);
        if (l == 0) break;
        // delta_{l-1} = (delta W_l) * silu'(Z_{l-1})
        float *nd = bufs[l & 1];
        gemm(s, (int)B, nin, dn, delta, dn, 0, w + L.W[l], nin, 0, nd, nin);
        hipLaunchKernelGGL(k_dsilu_mul, dim3(blocks(B * nin)), dim3(256), 0, s, B * nin, nd, wk.Z[l - 1]);
        delta = nd;
        dn = nin;
    }
    (void)hipMemsetAsync(grad + L.scale, 0, 10 * sizeof(float), s);
    return hip_ok("mlp grad");
}

extern "C" int fr_mlp_adam(int H, float *w, const float *grad, float *m, float *v, int step, float lr, void *stream) {
    if (H < 1 || !w || !grad || !m || !v || step < 1) return FR_DVM_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int64_t n = (int64_t)layout(H).scale;  // network weights only
    float c1 = 1.f - powf(0.9f, (float)step), c2 = 1.f - powf(0.999f, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(blocks(n)), dim3(256), 0, s, n, w, grad, m, v, c1, c2, lr);
    return hip_ok("adam");
}
