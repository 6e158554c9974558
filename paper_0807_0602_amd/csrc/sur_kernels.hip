// HIP kernels for gfx950 of the surrogate network: a multilayer perceptron with d_in inputs,
// `depth` hidden SiLU layers of `width` units and 2 linear outputs, trained with an
// output-weighted mean squared error and Adam.
//
// Precision: the hidden-to-hidden layers run on MFMA (v_mfma_f32_16x16x32_bf16) with BF16
// weights and activations and FP32 accumulation, forward and backward.  The first layer (a few
// inputs) and the output layer (2 outputs) run in FP32, so that the input features and the
// predicted front positions keep FP32 resolution.  Master weights, gradients and Adam moments
// are FP32; Adam refreshes BF16 copies of each hidden weight matrix and of its transpose.
//
// All reductions (bias and output-layer gradients, loss, data statistics) use fixed-order trees,
// so repeated runs give identical results.
#include "sur_internal.h"

namespace scf {
namespace sur {
namespace {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float sigmoid(float z) { return 1.0f / (1.0f + expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigmoid(z); }
__device__ __forceinline__ float silu_prime(float z) {
    const float s = sigmoid(z);
    return s * (1.0f + z * (1.0f - s));
}

// SplitMix64 output function (published constants): counter-based random numbers.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

constexpr int kThreads = 256;
// Predictions of up to this many rows per CU take 16 rows per block; so do training batches of 256 units,
// and of 128, whose blocks have half the threads, of twice as many.
constexpr int64_t kRows16 = 16;

// Fixed-order block reduction (kThreads threads).
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* sh) {
    const int tid = threadIdx.x;
    sh[tid] = v;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (tid < s) sh[tid] += sh[tid + s];
        __syncthreads();
    }
    const T r = sh[0];
    __syncthreads();
    return r;
}

// ---------------------------------------------------------------------------------------------
// MFMA GEMM, "NT" form: C[m][n] = sum_k A[m*lda + k] * B[n*ldb + k], BF16 operands contiguous in
// k, FP32 accumulation.  One wave per 16 x 16 output tile, four waves per block along n.
// Lane l holds A[m0 + l%16][k0 + 8(l/16) .. +7] and B[n0 + l%16][k0 + 8(l/16) .. +7] and receives
// C[m0 + 4(l/16) + i][n0 + l%16], i = 0..3 (layout checked on the device by the GEMM tests).
// M, N multiples of 16 (N of 64 per block row), K multiple of 32.  With FRAG, B is stored in
// fragment order (frag_at) instead: a weight matrix, whose row-major tiles would be read as 16
// half lines per load.
// ---------------------------------------------------------------------------------------------
// Fragment order of an (N x K) operand: the 16 x 32 tiles one after the other along k, each as the
// 64 lanes' eight values.
__device__ __forceinline__ int64_t frag_at(int n, int k, int K) {
    return ((int64_t)(n >> 4) * (K >> 5) + (k >> 5)) * 512 + (((k & 31) >> 3) * 16 + (n & 15)) * 8 + (k & 7);
}

template <bool FRAG, class Epi>
__global__ void __launch_bounds__(256)
k_gemm_nt(const __bf16* __restrict__ A, int lda, const __bf16* __restrict__ B, int ldb, int K,
          Epi epi) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int m0 = blockIdx.x * 16;
    const int n0 = (blockIdx.y * 4 + wave) * 16;
    const int r = lane & 15, g = lane >> 4;
    const __bf16* a = A + (int64_t)(m0 + r) * lda + 8 * g;
    const __bf16* b = FRAG ? B + (int64_t)(n0 >> 4) * (K >> 5) * 512 + 8 * lane : B + (int64_t)(n0 + r) * ldb + 8 * g;
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = 0; k0 < K; k0 += 32) {
        const bf8 fa = *reinterpret_cast<const bf8*>(a + k0);
        const bf8 fb = *reinterpret_cast<const bf8*>(b + (FRAG ? 16 * k0 : k0));
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, acc, 0, 0, 0);
    }
    epi(m0 + 4 * g, n0 + r, acc);
}

// Forward hidden layer: z = acc + bias; keeps z (FP32) for the backward pass and h = silu(z) in
// BF16, both row-major [m][n] and transposed [n][m] (the transposed copy feeds the weight
// gradient, which reduces over m).
struct EpiForward {
    const float* bias;
    float* Z;           // [M][N]
    __bf16* H;          // [M][N]
    __bf16* HT;         // [N][M]
    int N, M;
    __device__ void operator()(int mrow, int n, f4 acc) const {
        bf4 t;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float z = acc[i] + bias[n];
            Z[(int64_t)(mrow + i) * N + n] = z;
            const __bf16 h = (__bf16)silu(z);
            H[(int64_t)(mrow + i) * N + n] = h;
            t[i] = h;
        }
        *reinterpret_cast<bf4*>(HT + (int64_t)n * M + mrow) = t;
    }
};

// Back-propagation through a hidden layer: acc = dH of the layer below; dz = dH * silu'(z).
struct EpiBackward {
    const float* Zprev;   // [M][N] pre-activations of the layer below
    float* dZ;            // [M][N] FP32 (bias gradient, first-layer weight gradient)
    __bf16* dZb;          // [M][N]
    __bf16* dZbT;         // [N][M]
    int N, M;
    __device__ void operator()(int mrow, int n, f4 acc) const {
        bf4 t;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t o = (int64_t)(mrow + i) * N + n;
            const float dz = acc[i] * silu_prime(Zprev[o]);
            dZ[o] = dz;
            const __bf16 hb = (__bf16)dz;
            dZb[o] = hb;
            t[i] = hb;
        }
        *reinterpret_cast<bf4*>(dZbT + (int64_t)n * M + mrow) = t;
    }
};

// Weight gradient: dW[n_out][k_in] = acc.
struct EpiWeightGrad {
    float* dW;
    int N;
    __device__ void operator()(int mrow, int n, f4 acc) const {
#pragma unroll
        for (int i = 0; i < 4; ++i) dW[(int64_t)(mrow + i) * N + n] = acc[i];
    }
};

// ---------------------------------------------------------------------------------------------
// First layer (FP32): z = Xn W1^T + b1, one thread per (row, unit).
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads)
k_first_forward(const float* __restrict__ X, int d_in, const float* __restrict__ W,
                const float* __restrict__ bias, int width, int rows, float* __restrict__ Z,
                __bf16* __restrict__ H, __bf16* __restrict__ HT) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= (int64_t)rows * width) return;
    const int m = (int)(i / width), n = (int)(i % width);
    float z = bias[n];
    for (int k = 0; k < d_in; ++k) z += X[(int64_t)m * d_in + k] * W[n * d_in + k];
    Z[i] = z;
    const __bf16 h = (__bf16)silu(z);
    H[i] = h;
    HT[(int64_t)n * rows + m] = h;
}

// First-layer gradients: dW1[n][k] = sum_m dZ1[m][n] Xn[m][k], db1[n] = sum_m dZ1[m][n].
// One block per unit n; one fixed-order reduction per input (k = d_in gives the bias).
__global__ void __launch_bounds__(kThreads)
k_first_grad(const float* __restrict__ dZ, const float* __restrict__ X, int d_in, int width,
             int rows, float* __restrict__ dW, float* __restrict__ db) {
    __shared__ float sh[kThreads];
    const int n = blockIdx.x;
    for (int k = 0; k <= d_in; ++k) {
        float a = 0.0f;
        for (int m = threadIdx.x; m < rows; m += kThreads)
            a += dZ[(int64_t)m * width + n] * (k < d_in ? X[(int64_t)m * d_in + k] : 1.0f);
        a = block_sum(a, sh);
        if (threadIdx.x == 0) {
            if (k < d_in) dW[n * d_in + k] = a;
            else db[n] = a;
        }
    }
}

// Column sums of an FP32 [rows][width] matrix (bias gradients), one block per column.
__global__ void __launch_bounds__(kThreads)
k_colsum(const float* __restrict__ M, int width, int rows, float* __restrict__ out) {
    __shared__ float sh[kThreads];
    const int n = blockIdx.x;
    float a = 0.0f;
    for (int m = threadIdx.x; m < rows; m += kThreads) a += M[(int64_t)m * width + n];
    a = block_sum(a, sh);
    if (threadIdx.x == 0) out[n] = a;
}

// ---------------------------------------------------------------------------------------------
// Output layer, loss and the first backward step, one wave per row:
//   y_o = b_o + sum_k silu(z_k) W_o[k];  r = y - t;  loss_m = w_m |r|^2 / 2;  dy = w_m r / n
// (n = number of real rows; padding rows carry w = 0)
//   dz_k = (sum_o dy_o W_o[k]) silu'(z_k)  -> dZ (FP32), dZb, dZbT (BF16) of the last layer.
// With T == nullptr only y is computed (inference).
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads)
k_output(const float* __restrict__ Z, int width, int rows, const float* __restrict__ W,
         const float* __restrict__ bias, const float* __restrict__ T, const float* __restrict__ w,
         float inv_n, float* __restrict__ Y, float* __restrict__ dY, float* __restrict__ rowloss,
         float* __restrict__ dZ, __bf16* __restrict__ dZb, __bf16* __restrict__ dZbT) {
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (m >= rows) return;
    const float* z = Z + (int64_t)m * width;
    float s0 = 0.0f, s1 = 0.0f;
    for (int k = lane; k < width; k += 64) {
        const float h = silu(z[k]);
        s0 += h * W[k];
        s1 += h * W[width + k];
    }
    for (int off = 32; off > 0; off >>= 1) {
        s0 += __shfl_xor(s0, off);
        s1 += __shfl_xor(s1, off);
    }
    const float y0 = s0 + bias[0], y1 = s1 + bias[1];
    if (lane == 0) {
        Y[2 * m] = y0;
        Y[2 * m + 1] = y1;
    }
    if (!T) return;
    const float r0 = y0 - T[2 * m], r1 = y1 - T[2 * m + 1];
    const float wm = w[m];
    const float d0 = wm * r0 * inv_n, d1 = wm * r1 * inv_n;
    if (lane == 0) {
        dY[2 * m] = d0;
        dY[2 * m + 1] = d1;
        rowloss[m] = 0.5f * wm * (r0 * r0 + r1 * r1);
    }
    for (int k = lane; k < width; k += 64) {
        const float dz = (d0 * W[k] + d1 * W[width + k]) * silu_prime(z[k]);
        dZ[(int64_t)m * width + k] = dz;
        dZb[(int64_t)m * width + k] = (__bf16)dz;
        dZbT[(int64_t)k * rows + m] = (__bf16)dz;
    }
}

// Output-layer gradients: dW_o[k] = sum_m dy_o silu(z_mk), db_o = sum_m dy_o; block per k
// (block `width` computes the bias gradient).
__global__ void __launch_bounds__(kThreads)
k_output_grad(const float* __restrict__ Z, int width, int rows, const float* __restrict__ dY,
              float* __restrict__ dW, float* __restrict__ db) {
    __shared__ float sh[kThreads];
    const int k = blockIdx.x;
    float a0 = 0.0f, a1 = 0.0f;
    for (int m = threadIdx.x; m < rows; m += kThreads) {
        const float h = k < width ? silu(Z[(int64_t)m * width + k]) : 1.0f;
        a0 += dY[2 * m] * h;
        a1 += dY[2 * m + 1] * h;
    }
    a0 = block_sum(a0, sh);
    a1 = block_sum(a1, sh);
    if (threadIdx.x == 0) {
        if (k < width) {
            dW[k] = a0;
            dW[width + k] = a1;
        } else {
            db[0] = a0;
            db[1] = a1;
        }
    }
}

// Sum of the per-row losses (fixed order, one block).
__global__ void __launch_bounds__(kThreads)
k_loss_sum(const float* __restrict__ rowloss, int rows, float inv_n, float* __restrict__ out) {
    __shared__ double sh[kThreads];
    double a = 0.0;
    for (int m = threadIdx.x; m < rows; m += kThreads) a += (double)rowloss[m];
    a = block_sum(a, sh);
    if (threadIdx.x == 0) out[0] = (float)(a * inv_n);
}

// ---------------------------------------------------------------------------------------------
// Adam (Kingma and Ba, 2015) with bias correction; the step count and the learning rate live on
// the device so that captured graphs advance the one and follow changes of the other.  Hidden weight matrices are copied to BF16, row-major and
// transposed.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads)
k_adam(float* __restrict__ theta, const float* __restrict__ grad, float* __restrict__ m1,
       float* __restrict__ m2, int64_t n, const int64_t* __restrict__ step,
       const float* __restrict__ lr_dev, float b1, float b2, float eps) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const float lr = *lr_dev;
    const float t = (float)(*step + 1);
    const float g = grad[i];
    const float a = b1 * m1[i] + (1.0f - b1) * g;
    const float v = b2 * m2[i] + (1.0f - b2) * g * g;
    m1[i] = a;
    m2[i] = v;
    const float ah = a / (1.0f - powf(b1, t));
    const float vh = v / (1.0f - powf(b2, t));
    theta[i] -= lr * ah / (sqrtf(vh) + eps);
}

__global__ void k_bump64(int64_t* c) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *c = *c + 1;
}

// BF16 copies of one (n_out x n_in) FP32 weight matrix and of its transpose, both in fragment order
// (frag_at).
__global__ void __launch_bounds__(kThreads)
k_shadow(const float* __restrict__ W, int n_out, int n_in, __bf16* __restrict__ Wb,
         __bf16* __restrict__ WbT) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= (int64_t)n_out * n_in) return;
    const int o = (int)(i / n_in), k = (int)(i % n_in);
    const __bf16 v = (__bf16)W[i];
    Wb[frag_at(o, k, n_in)] = v;
    WbT[frag_at(k, o, n_out)] = v;
}

// ---------------------------------------------------------------------------------------------
// Data: feature statistics (mean, standard deviation, min, max per input; FP64 sums, one block
// per feature), normalisation of an explicit batch, and random minibatches of the stored set.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads)
k_stats(const float* __restrict__ X, int d_in, int64_t n, float* __restrict__ mean,
        float* __restrict__ stdv, float* __restrict__ lo, float* __restrict__ hi) {
    __shared__ double sh[kThreads];
    __shared__ float sf[kThreads];
    const int k = blockIdx.x;
    double s = 0.0;
    float mn = INFINITY, mx = -INFINITY;
    for (int64_t m = threadIdx.x; m < n; m += kThreads) {
        const float v = X[m * d_in + k];
        s += v;
        mn = fminf(mn, v);
        mx = fmaxf(mx, v);
    }
    const double mu = block_sum(s, sh) / (double)n;
    double q = 0.0;
    for (int64_t m = threadIdx.x; m < n; m += kThreads) {
        const double d = X[m * d_in + k] - mu;
        q += d * d;
    }
    const double var = block_sum(q, sh) / (double)n;
    // min / max by the same fixed tree
    sf[threadIdx.x] = mn;
    __syncthreads();
    for (int st = kThreads / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st) sf[threadIdx.x] = fminf(sf[threadIdx.x], sf[threadIdx.x + st]);
        __syncthreads();
    }
    const float gmn = sf[0];
    __syncthreads();
    sf[threadIdx.x] = mx;
    __syncthreads();
    for (int st = kThreads / 2; st > 0; st >>= 1) {
        if (threadIdx.x < st) sf[threadIdx.x] = fmaxf(sf[threadIdx.x], sf[threadIdx.x + st]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        mean[k] = (float)mu;
        stdv[k] = var > 0.0 ? (float)sqrt(var) : 1.0f;
        lo[k] = gmn;
        hi[k] = sf[0];
    }
}

// Normalise rows of X into Xn (and copy targets / weights when given).  With rng set, row i is
// drawn from the stored set (src_rows rows) by a counter-based hash of (seed, step, i).
__global__ void __launch_bounds__(kThreads)
k_gather(const float* __restrict__ X, const float* __restrict__ T, const float* __restrict__ w,
         int64_t src_rows, int d_in, int rows, const float* __restrict__ mean,
         const float* __restrict__ stdv, float* __restrict__ Xn, float* __restrict__ Tb,
         float* __restrict__ wb, int rng, uint64_t seed, const int64_t* __restrict__ step) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= rows) return;
    int64_t j = i;
    if (rng) {
        const uint64_t h = mix64(seed ^ mix64((uint64_t)(*step) * 0x100000001B3ull + (uint64_t)i));
        j = (int64_t)(h % (uint64_t)src_rows);
    }
    for (int k = 0; k < d_in; ++k) Xn[(int64_t)i * d_in + k] = (X[j * d_in + k] - mean[k]) / stdv[k];
    if (Tb) {
        Tb[2 * i] = T[2 * j];
        Tb[2 * i + 1] = T[2 * j + 1];
        wb[i] = w[j];
    }
}

// Rows i < n of X (caller's device memory) normalised into Xn as k_gather does; padding rows
// [n, rows) are set to 0 (rows are independent through the network and their outputs unused).
__global__ void __launch_bounds__(kThreads)
k_normalise(const float* __restrict__ X, int64_t n, int d_in, int rows, const float* __restrict__ mean,
            const float* __restrict__ stdv, float* __restrict__ Xn) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= rows) return;
    for (int k = 0; k < d_in; ++k)
        Xn[(int64_t)i * d_in + k] = i < n ? (X[(int64_t)i * d_in + k] - mean[k]) / stdv[k] : 0.0f;
}

__global__ void __launch_bounds__(kThreads) k_fill_u8(uint8_t* __restrict__ p, int64_t n, uint8_t v) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void __launch_bounds__(kThreads)
k_copy_u8(uint8_t* __restrict__ to, const uint8_t* __restrict__ from, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) to[i] = from[i];
}

// Inputs inside the axis-aligned box of the stored training inputs.
__global__ void __launch_bounds__(kThreads)
k_hull(const float* __restrict__ X, int d_in, int rows, const float* __restrict__ lo,
       const float* __restrict__ hi, uint8_t* __restrict__ in) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= rows) return;
    uint8_t ok = 1;
    for (int k = 0; k < d_in; ++k) {
        const float v = X[(int64_t)i * d_in + k];
        if (!(v >= lo[k] && v <= hi[k])) ok = 0;
    }
    in[i] = ok;
}

// Parameter initialisation: W uniform in +-1/sqrt(fan_in) from a counter-based hash, b = 0.
__global__ void __launch_bounds__(kThreads)
k_init_params(float* __restrict__ theta, int64_t off, int n_out, int n_in, uint64_t seed) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t nw = (int64_t)n_out * n_in;
    if (i >= nw + n_out) return;
    float v = 0.0f;
    if (i < nw) {
        const uint64_t h = mix64(seed ^ mix64((uint64_t)(off + i)));
        const float u = (float)(h >> 40) * (1.0f / 16777216.0f);   // [0, 1)
        v = (2.0f * u - 1.0f) / sqrtf((float)n_in);
    }
    theta[off + i] = v;
}

// ---------------------------------------------------------------------------------------------
// Whole-network kernels.  A block takes a few rows through every layer: the activations stay in
// LDS (BF16, the next layer's A operand) and only the weights are read again, from L2.  The layer
// kernels above spend a launch per layer and write pre-activations and two copies of the
// activations to memory, of which a prediction needs nothing and a training step only what the
// weight gradients read.  Each value is computed by the same operations in the same order as
// there, so the results are the same bit for bit.
// ---------------------------------------------------------------------------------------------
// A wave owns 16 NT units; its slice of a layer's weights sits in NT W / 8 registers.
template <int W, int NT>
struct Slice {
    bf8 k[NT][W / 32];
    __device__ __forceinline__ void load(const __bf16* __restrict__ Wl, int n0) {
        const __bf16* b = Wl + (int64_t)n0 * W + 8 * (threadIdx.x & 63);   // fragment order
#pragma unroll
        for (int j = 0; j < W / 32; ++j)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) k[nt][j] = *reinterpret_cast<const bf8*>(b + nt * 16 * W + 512 * j);
    }
};

// acc[mt][nt] = rows 16 mt .. of the block's activations hb (LDS, row stride W + 8: eight lanes'
// 16-byte reads fall on different banks) times the wave's slice, units 16 nt ...
template <int W, int MT, int NT>
__device__ __forceinline__ void layer_mma(const __bf16* hb, const Slice<W, NT>& b, f4 (&acc)[MT][NT]) {
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < W / 32; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const bf8 a = *reinterpret_cast<const bf8*>(hb + (mt * 16 + r) * (W + 8) + 32 * j + 8 * g);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b.k[nt][j], acc[mt][nt], 0, 0, 0);
        }
}

// First layer (FP32) in the same tiles: acc = xs W1^T + b1 with xs the block's normalised rows and
// w1 the layer's weights (LDS).
template <int MT, int NT>
__device__ __forceinline__ void layer_first(const float (*xs)[kMaxIn + 1], int d_in, const float* w1,
                                            const float* __restrict__ b1, int u, f4 (&acc)[MT][NT]) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const float bias = b1[u + 16 * nt];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = f4{bias, bias, bias, bias};
    }
    for (int k = 0; k < d_in; ++k)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const float w = w1[(u + 16 * nt) * d_in + k];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[mt][nt][i] += xs[mt * 16 + 4 * g + i][k] * w;
        }
}

// One row of the output layer by one wave: h (LDS, FP32 activations) times the two output rows,
// summed as k_output sums them.
template <int W>
__device__ __forceinline__ void output_row(const float* h, const float* __restrict__ Wo, float& s0, float& s1) {
    const int lane = threadIdx.x & 63;
    s0 = 0.0f;
    s1 = 0.0f;
#pragma unroll
    for (int k = lane; k < W; k += 64) {
        s0 += h[k] * Wo[k];
        s1 += h[k] * Wo[W + k];
    }
    for (int off = 32; off > 0; off >>= 1) {
        s0 += __shfl_xor(s0, off);
        s1 += __shfl_xor(s1, off);
    }
}

// Prediction: rows [n] of X (raw inputs) to Y and, with `in`, the hull test (`hull` 0: all
// outside).  16 MT rows per block of W / (16 NT) waves.  The first and last layers' weights wait in
// LDS with the inputs, so that one trip to memory comes before the first barrier and only the
// hidden layers' slices after it.  Bound by that chain for few rows (a block's 20 000 cycles: 3600
// to the inputs, 4400 per hidden layer, half of it the weights' way from L2) and by the vector
// work of SiLU for many (about 28 instructions per unit, exp and an IEEE division).  256 x 4, 5
// inputs: 2048 device rows 10.1 us, for 35.9 with a launch per layer; 32064 rows 53 us, for 8 x
// 62 us.  Weights in fragment order instead of row-major: 2250 cycles to load a layer for 7700.
template <int W, int MT, int NT>
__global__ void __launch_bounds__(4 * W / NT)
k_predict(const float* __restrict__ X, int64_t n, int d_in, int depth, const float* __restrict__ mean,
          const float* __restrict__ stdv, const float* __restrict__ lo, const float* __restrict__ hi, int hull,
          const float* __restrict__ theta, const __bf16* __restrict__ Wb, float* __restrict__ Y,
          uint8_t* __restrict__ in) {
    constexpr int T = 4 * W / NT, M = 16 * MT, LDF = W + 4;
    __shared__ __align__(16) float sh[M * LDF];   // first-layer weights, BF16 activations, FP32 ones
    __shared__ float wo[2 * W + 2];
    __shared__ float xs[M][kMaxIn + 1];
    __shared__ uint8_t ok[M][kMaxIn];
    __bf16* hb = reinterpret_cast<__bf16*>(sh);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
    const int64_t m0 = (int64_t)blockIdx.x * M;
    const int n0 = wave * 16 * NT, u = n0 + r;
    const float* bias = theta + (int64_t)W * d_in;   // biases of the current layer
    const float* out = bias + (int64_t)depth * W + (int64_t)(depth - 1) * W * W;
    Slice<W, NT> b, next;
    if (depth > 1) b.load(Wb, n0);
    float* w1 = sh;
    const bool staged = W * d_in <= M * LDF;
    if (staged)
        for (int i = tid; i < W * d_in; i += T) w1[i] = theta[i];
    for (int i = tid; i < 2 * W + 2; i += T) wo[i] = out[i];
    for (int i = tid; i < M * d_in; i += T) {
        const int m = i / d_in, k = i % d_in;
        const float v = m0 + m < n ? X[(m0 + m) * d_in + k] : 0.0f;
        xs[m][k] = m0 + m < n ? (v - mean[k]) / stdv[k] : 0.0f;
        ok[m][k] = v >= lo[k] && v <= hi[k];
    }
    __syncthreads();
    if (in && tid < M && m0 + tid < n) {
        uint8_t all = hull ? 1 : 0;
        for (int k = 0; k < d_in; ++k) all &= ok[tid][k];
        in[m0 + tid] = all;
    }
    f4 acc[MT][NT];
    layer_first<MT, NT>(xs, d_in, staged ? w1 : theta, bias, u, acc);
    __syncthreads();
    for (int l = 0; l + 1 < depth; ++l) {
        // one unit tile per wave leaves the registers to load a layer ahead
        if (NT == 1 && l + 2 < depth) next.load(Wb + (int64_t)(l + 1) * W * W, n0);
        bias += W + (int64_t)W * W;
        float add[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) add[nt] = bias[u + 16 * nt];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    hb[(mt * 16 + 4 * g + i) * (W + 8) + u + 16 * nt] = (__bf16)silu(acc[mt][nt][i]);
        __syncthreads();
        layer_mma<W, MT, NT>(hb, b, acc);
        if (NT == 1) b = next;
        else if (l + 2 < depth) b.load(Wb + (int64_t)(l + 1) * W * W, n0);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[mt][nt][i] += add[nt];
        __syncthreads();
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) sh[(mt * 16 + 4 * g + i) * LDF + u + 16 * nt] = silu(acc[mt][nt][i]);
    __syncthreads();
    for (int m = wave; m < M; m += T / 64) {
        float s0, s1;
        output_row<W>(sh + m * LDF, wo, s0, s1);
        if (lane == 0 && m0 + m < n) {
            Y[2 * (m0 + m)] = s0 + wo[2 * W];
            Y[2 * (m0 + m) + 1] = s1 + wo[2 * W + 1];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// A training step in two launches.  k_train_rows takes 16 or 32 rows through the forward pass, the loss
// and the backward pass, keeping silu'(z) of every layer in registers (at 256 x 4, the most it takes, 30
// of the 128 spill with 32 rows per block and 3 with 16; elsewhere none); it writes what the weight
// gradients read: both transposed BF16 operands of every hidden layer, the FP32 dz of every layer
// and the last activations.  k_train_grads reduces them over the batch, one block per 32 x 32 tile
// of a hidden matrix or 16 columns of a sum, and applies Adam to what it has just summed (or
// writes the gradient).  Every sum keeps the order of the layer kernels: a tile's products run
// through the whole batch in one accumulator, a column's rows in 256 interleaved chains and a tree.
// Measured, 256 x 4 with 5 inputs and 8192 rows: 42 + 38 us, for 28 launches and 594 us.  The first
// is bound by its chain of barriers, one block of 16 waves per CU, in the forward half, and in the
// backward half by the 65 MB it writes; the second by what it reads from beyond L2 and the time a
// trip there takes (61 MB with tiles and sums dealt to the XCDs by operand, 44 us in block order).
// Where 16 rows per block fill the CUs no more than once, the chain is shorter with them: us per step
// with 32 and with 16, 256 x 4: 64 rows 43.8 and 30.7, 1024 49.1 and 36.1, 4096 62.4 and 49.3, 6144
// 73.4 and 75.0; 128 x 3: 64 rows 22.6 and 19.2, 4096 40.5 and 37.4, 8192 48.2 and 47.1.
// ---------------------------------------------------------------------------------------------
struct TrainData {
    const float *X, *T, *w;   // stored rows
    int64_t src_rows;
    int d_in, rng;            // rng: rows drawn by the hash of (seed, step, row), else row i itself
    const float *mean, *stdv;
    uint64_t seed;
    int64_t* step;            // [0] steps done, [1] the step in progress
};

template <int W, int D, int MT>
__global__ void __launch_bounds__(4 * W)
k_train_rows(const TrainData d, const float* __restrict__ theta, const __bf16* __restrict__ Wb,
             const __bf16* __restrict__ WbT, int rows, float inv_n, TrainWork wk) {
    constexpr int T = 4 * W, M = 16 * MT, LDF = W + 4;
    __shared__ __align__(16) float sh[32 * LDF];   // first-layer weights, BF16 operands, FP32 activations
    __shared__ float xs[M][kMaxIn + 1];
    __shared__ float wo[2 * W + 2], dy[M][2], tw[M][3];
    __shared__ int64_t row[M];
    __bf16* hb = reinterpret_cast<__bf16*>(sh);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
    const int m0 = blockIdx.x * M, n0 = wave * 16, u = n0 + r, din = d.d_in;
    const int64_t plane = (int64_t)rows * W;
    const float* bias = theta + (int64_t)W * din;
    const float* out = bias + (int64_t)D * W + (int64_t)(D - 1) * W * W;
    Slice<W, 1> b, next;
    if (D > 1) b.load(Wb, n0);
    if (tid < M) {
        const int i = m0 + tid;
        int64_t j = i;
        if (d.rng) {
            const uint64_t h = mix64(d.seed ^ mix64((uint64_t)(*d.step) * 0x100000001B3ull + (uint64_t)i));
            j = (int64_t)(h % (uint64_t)d.src_rows);
        }
        row[tid] = j;
        tw[tid][0] = d.T[2 * j];
        tw[tid][1] = d.T[2 * j + 1];
        tw[tid][2] = d.w[j];
        if (i == 0) d.step[1] = d.step[0] + 1;
    }
    const bool staged = W * din <= 32 * LDF;
    if (staged)
        for (int i = tid; i < W * din; i += T) sh[i] = theta[i];
    for (int i = tid; i < 2 * W + 2; i += T) wo[i] = out[i];
    __syncthreads();
    for (int i = tid; i < M * din; i += T) {
        const int m = i / din, k = i % din;
        const float v = (d.X[row[m] * din + k] - d.mean[k]) / d.stdv[k];
        xs[m][k] = v;
        wk.Xn[(int64_t)(m0 + m) * din + k] = v;
    }
    __syncthreads();
    f4 acc[MT][1], sp[D][MT];
    layer_first<MT, 1>(xs, din, staged ? sh : theta, bias, u, acc);
    __syncthreads();
#pragma unroll
    for (int l = 0; l < D; ++l) {
        const bool last = l == D - 1;
        if (l + 2 < D) next.load(Wb + (int64_t)(l + 1) * W * W, n0);
        else if (l + 2 == D) next.load(WbT + (int64_t)(D - 2) * W * W, n0);   // first backward product
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            bf4 t;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float z = acc[mt][0][i], s = sigmoid(z), h = z * s;
                sp[l][mt][i] = s * (1.0f + z * (1.0f - s));
                const int m = mt * 16 + 4 * g + i;
                if (last) {
                    sh[m * LDF + u] = h;
                } else {
                    t[i] = (__bf16)h;
                    hb[m * (W + 8) + u] = t[i];
                }
            }
            if (!last) *reinterpret_cast<bf4*>(wk.HT + l * plane + (int64_t)u * rows + m0 + mt * 16 + 4 * g) = t;
        }
        __syncthreads();
        if (last) break;
        layer_mma<W, MT, 1>(hb, b, acc);
        b = next;
        bias += W + (int64_t)W * W;
        const float add = bias[u];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[mt][0][i] += add;
        __syncthreads();
    }
    for (int m = wave; m < M; m += T / 64) {
        float s0, s1;
        const float* h = sh + m * LDF;
        output_row<W>(h, wo, s0, s1);
        for (int k = lane; k < W; k += 64) wk.Hlast[(int64_t)(m0 + m) * W + k] = h[k];
        const float y0 = s0 + wo[2 * W], y1 = s1 + wo[2 * W + 1];
        const float r0 = y0 - tw[m][0], r1 = y1 - tw[m][1];
        const float wm = tw[m][2];
        const float d0 = wm * r0 * inv_n, d1 = wm * r1 * inv_n;
        if (lane == 0) {
            dy[m][0] = d0;
            dy[m][1] = d1;
            wk.dY[2 * (m0 + m)] = d0;
            wk.dY[2 * (m0 + m) + 1] = d1;
            wk.rowloss[m0 + m] = 0.5f * wm * (r0 * r0 + r1 * r1);
        }
    }
    __syncthreads();
#pragma unroll
    for (int l = D - 1; l >= 0; --l) {
        if (l < D - 1) {
            layer_mma<W, MT, 1>(hb, b, acc);   // dh of layer l
            b = next;
            __syncthreads();
        }
        if (l >= 2) next.load(WbT + (int64_t)(l - 2) * W * W, n0);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            bf4 t;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = mt * 16 + 4 * g + i;
                const float dh = l == D - 1 ? dy[m][0] * wo[u] + dy[m][1] * wo[W + u] : acc[mt][0][i];
                const float dz = dh * sp[l][mt][i];
                wk.dZ[l * plane + (int64_t)(m0 + m) * W + u] = dz;
                t[i] = (__bf16)dz;
                if (l > 0) hb[m * (W + 8) + u] = t[i];
            }
            if (l > 0) *reinterpret_cast<bf4*>(wk.dZT + l * plane + (int64_t)u * rows + m0 + mt * 16 + 4 * g) = t;
        }
        if (l > 0) __syncthreads();
    }
}

struct AdamArgs {
    float *theta, *m1, *m2, *grad;   // grad: written instead of an update when update == 0
    const int64_t* step;             // [1]: the step in progress
    const float* lr;
    float b1, b2, eps;
    int update;
};

__device__ __forceinline__ float adam_one(const AdamArgs& a, int64_t i, float g, float lr, float c1, float c2) {
    const float m = a.b1 * a.m1[i] + (1.0f - a.b1) * g;
    const float v = a.b2 * a.m2[i] + (1.0f - a.b2) * g * g;
    a.m1[i] = m;
    a.m2[i] = v;
    const float ah = m / c1;
    const float vh = v / c2;
    float th = a.theta[i];
    th -= lr * ah / (sqrtf(vh) + a.eps);
    a.theta[i] = th;
    return th;
}

// Sum over the batch of NV values per (row, column), 16 columns and 16 classes of rows per block:
// the thread of class c sums the rows c + 16 j (mod 256) in chain j, the chains are combined as a
// tree over the 256 chains would (j and j + 8 first), then the classes.  `load` fetches a row's
// values and `add` adds them; the loads of U x 16 rows are issued together (the rows come from
// beyond L2 at 2-3 us a trip; with 16 in flight the sums took 139 us of a 8192-row step).
template <int NV, int U, class V, class L, class A>
__device__ __forceinline__ void column_sums(int rows, L load, A add, float (&sum)[NV], float (*sh)[16][NV]) {
    const int c = threadIdx.x & 15, cls = threadIdx.x >> 4;
    float a[16][NV];
#pragma unroll
    for (int j = 0; j < 16; ++j)
#pragma unroll
        for (int q = 0; q < NV; ++q) a[j][q] = 0.0f;
    int m = cls;
    for (const int end = rows - (rows % (256 * U)); m < end; m += 256 * U) {
        V v[U][16];
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int j = 0; j < 16; ++j) v[k][j] = load(m + 256 * k + 16 * j);
        __builtin_amdgcn_sched_barrier(0);   // or the loads are spread over the sums again
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int j = 0; j < 16; ++j) add(a[j], v[k][j]);
    }
    for (; m < rows; m += 256)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (m + 16 * j < rows) add(a[j], load(m + 16 * j));
#pragma unroll
    for (int s = 8; s > 0; s >>= 1)
#pragma unroll
        for (int j = 0; j < s; ++j)
#pragma unroll
            for (int q = 0; q < NV; ++q) a[j][q] += a[j + s][q];
#pragma unroll
    for (int q = 0; q < NV; ++q) sh[cls][c][q] = a[0][q];
    __syncthreads();
    for (int s = 8; s > 0; s >>= 1) {
        if (cls < s)
#pragma unroll
            for (int q = 0; q < NV; ++q) sh[cls][c][q] += sh[cls + s][c][q];
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) sum[q] = sh[0][c][q];
}

// Blocks: (D - 1) (W / 32)^2 tiles of the hidden matrices; W / 16 column groups for each of the
// d_in + 1 first-layer sums, the D - 1 hidden biases and the output rows; one for the loss and the
// output biases.
template <int W>
__global__ void __launch_bounds__(256)
k_train_grads(int D, int d_in, int rows, float inv_n, TrainWork wk, AdamArgs ad, __bf16* __restrict__ Wb,
              __bf16* __restrict__ WbT, float* __restrict__ loss, int64_t* __restrict__ step) {
    constexpr int CH = 128, LD = CH + 8;   // eight lanes' 16-byte reads fall on different banks
    __shared__ __align__(16) __bf16 sa[2][32 * LD], sb[2][32 * LD];
    __shared__ float fs[16][16][2];
    __shared__ double ds[kThreads];
    __shared__ float corr[2];
    const int tid = threadIdx.x;
    if (ad.update && tid == 0) {
        const float t = (float)ad.step[1];
        corr[0] = 1.0f - powf(ad.b1, t);
        corr[1] = 1.0f - powf(ad.b2, t);
    }
    const float lr = *ad.lr;
    const int64_t plane = (int64_t)rows * W, hidden = (int64_t)W * W + W, first = (int64_t)W * d_in + W;
    constexpr int side = W / 32, groups = W / 16;
    const int tiles = (D - 1) * side * side;
    int blk = blockIdx.x;
    if (blk < tiles) {
        // an XCD (block b runs on XCD b mod 8) takes the same patch of every matrix, two tiles wide, and
        // so reads six of a layer's 16 operand strips through its L2; a column of tiles would be nine
        constexpr int PER = side * side / 8, KG = side / 2;
        const int x = blk & 7, i = blk >> 3, j = i % PER;
        const int l = 1 + i / PER, o0 = (x / KG * (PER / 2) + j / 2) * 32, k0 = (x % KG * 2 + (j & 1)) * 32;
        const int lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4, wm = (wave & 1) * 16, wn = (wave >> 1) * 16;
        // chunks of CH batch rows: a thread brings 32 bytes of one row of each operand
        const int row = tid >> 3, seg = (tid & 7) * 8;
        const __bf16* pa = wk.dZT + l * plane + (int64_t)(o0 + row) * rows + seg;
        const __bf16* pb = wk.HT + (l - 1) * plane + (int64_t)(k0 + row) * rows + seg;
        constexpr int PF = 2;   // chunks in flight
        const int nc = rows / CH;
        bf8 ra[PF][2], rb[PF][2];
        auto fetch = [&](int p, int c) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                ra[p][q] = *reinterpret_cast<const bf8*>(pa + CH * c + 64 * q);
                rb[p][q] = *reinterpret_cast<const bf8*>(pb + CH * c + 64 * q);
            }
        };
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        // one barrier per chunk: the buffer written next was read before the last barrier
        auto product = [&](int p, int n) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < n; j += 32) {
                const bf8 fa = *reinterpret_cast<const bf8*>(&sa[p][(wm + r) * LD + j + 8 * g]);
                const bf8 fb = *reinterpret_cast<const bf8*>(&sb[p][(wn + r) * LD + j + 8 * g]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, acc, 0, 0, 0);
            }
        };
        auto stage = [&](int p) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                *reinterpret_cast<bf8*>(&sa[p][row * LD + seg + 64 * q]) = ra[p][q];
                *reinterpret_cast<bf8*>(&sb[p][row * LD + seg + 64 * q]) = rb[p][q];
            }
        };
        int c0 = 0;
        if (nc > 0) {
#pragma unroll
            for (int p = 0; p < PF; ++p) fetch(p, min(p, nc - 1));
            for (; c0 + PF <= nc; c0 += PF)
#pragma unroll
                for (int p = 0; p < PF; ++p) {
                    stage(p);
                    // past the end the last chunk is loaded again: no branch, so the compiler keeps
                    // count of the loads in flight
                    fetch(p, min(c0 + p + PF, nc - 1));
                    product(p, CH);
                }
            if (c0 < nc) {
                stage(0);
                product(0, CH);
            }
        }
        if (rows % CH) {   // the last 64 rows
            const bf8 la = *reinterpret_cast<const bf8*>(pa + CH * nc), lb = *reinterpret_cast<const bf8*>(pb + CH * nc);
            __syncthreads();
            *reinterpret_cast<bf8*>(&sa[0][row * LD + seg]) = la;
            *reinterpret_cast<bf8*>(&sb[0][row * LD + seg]) = lb;
            product(0, 64);
        }
        const int64_t at = first + (l - 1) * hidden;
        const int o = o0 + wm + 4 * g, k = k0 + wn + r;
        bf4 t;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t q = at + (int64_t)(o + i) * W + k;
            if (!ad.update) {
                ad.grad[q] = acc[i];
                continue;
            }
            t[i] = (__bf16)adam_one(ad, q, acc[i], lr, corr[0], corr[1]);
            Wb[(l - 1) * (int64_t)W * W + frag_at(o + i, k, W)] = t[i];
        }
        if (ad.update) *reinterpret_cast<bf4*>(WbT + (l - 1) * (int64_t)W * W + frag_at(k, o, W)) = t;
        return;
    }
    blk -= tiles;
    __syncthreads();   // corr
    auto put = [&](int64_t q, float g) {
        if (!ad.update) ad.grad[q] = g;
        else (void)adam_one(ad, q, g, lr, corr[0], corr[1]);
    };
    const int c = tid & 15;
    // an XCD takes the same columns of every sum (the first layer's read the same dz)
    const int kind = (blk >> 3) / (groups / 8), n = ((blk & 7) * (groups / 8) + (blk >> 3) % (groups / 8)) * 16 + c;
    if (kind < d_in + D) {
        // first layer: inputs k < d_in and bias; then the biases of layers 1 .. D - 1
        float s[1];
        float (*sh)[16][1] = reinterpret_cast<float (*)[16][1]>(&fs[0][0][0]);
        if (kind < d_in) {
            const float* dz = wk.dZ + n;
            const float* x = wk.Xn + kind;
            struct V { float dz, x; };
            column_sums<1, 2, V>(rows, [&](int m) { return V{dz[(int64_t)m * W], x[(int64_t)m * d_in]}; },
                                 [](float (&a)[1], const V& v) { a[0] += v.dz * v.x; }, s, sh);
        } else {
            const float* dz = wk.dZ + (kind - d_in) * plane + n;
            column_sums<1, 4, float>(rows, [&](int m) { return dz[(int64_t)m * W]; },
                                     [](float (&a)[1], float v) { a[0] += v; }, s, sh);
        }
        if (tid < 16) {
            if (kind < d_in) put((int64_t)n * d_in + kind, s[0]);
            else if (kind == d_in) put((int64_t)W * d_in + n, s[0]);
            else put(first + (kind - d_in - 1) * hidden + (int64_t)W * W + n, s[0]);
        }
        return;
    }
    const int64_t out = first + (D - 1) * hidden;
    if (kind == d_in + D) {
        const int k = n;
        const float* h = wk.Hlast + k;
        const float* dy = wk.dY;
        float s[2];
        struct V { float h, d0, d1; };
        column_sums<2, 2, V>(rows, [&](int m) { return V{h[(int64_t)m * W], dy[2 * m], dy[2 * m + 1]}; },
                             [](float (&a)[2], const V& v) {
                                 a[0] += v.d0 * v.h;
                                 a[1] += v.d1 * v.h;
                             }, s, fs);
        if (tid < 16) {
            put(out + k, s[0]);
            put(out + W + k, s[1]);
        }
        return;
    }
    float* f = &fs[0][0][0];
    float b0 = 0.0f, b1 = 0.0f;
    double e = 0.0;
#pragma unroll 8
    for (int m = tid; m < rows; m += kThreads) {
        b0 += wk.dY[2 * m];
        b1 += wk.dY[2 * m + 1];
        e += (double)wk.rowloss[m];
    }
    b0 = block_sum(b0, f);
    b1 = block_sum(b1, f);
    e = block_sum(e, ds);
    if (tid == 0) {
        put(out + 2 * W, b0);
        put(out + 2 * W + 1, b1);
        loss[0] = (float)(e * inv_n);
        if (ad.update) step[0] = step[1];
    }
}

inline dim3 grid1(int64_t n) { return dim3((unsigned)((n + kThreads - 1) / kThreads)); }

}  // namespace

hipError_t gemm_forward(const __bf16* Hprev, const __bf16* Wb, const float* bias, int rows, int width,
                        float* Z, __bf16* H, __bf16* HT, hipStream_t s) {
    EpiForward epi{bias, Z, H, HT, width, rows};
    hipLaunchKernelGGL((k_gemm_nt<true, EpiForward>), dim3(rows / 16, width / 64), dim3(256), 0, s, Hprev,
                       width, Wb, width, width, epi);
    return hipGetLastError();
}

hipError_t gemm_backward(const __bf16* dZb, const __bf16* WbT, const float* Zprev, int rows,
                         int width, float* dZ, __bf16* dZbo, __bf16* dZbTo, hipStream_t s) {
    EpiBackward epi{Zprev, dZ, dZbo, dZbTo, width, rows};
    hipLaunchKernelGGL((k_gemm_nt<true, EpiBackward>), dim3(rows / 16, width / 64), dim3(256), 0, s, dZb,
                       width, WbT, width, width, epi);
    return hipGetLastError();
}

hipError_t gemm_weight_grad(const __bf16* dZbT, const __bf16* HT, int rows, int width, float* dW,
                            hipStream_t s) {
    EpiWeightGrad epi{dW, width};
    hipLaunchKernelGGL((k_gemm_nt<false, EpiWeightGrad>), dim3(width / 16, width / 64), dim3(256), 0, s, dZbT,
                       rows, HT, rows, rows, epi);
    return hipGetLastError();
}

hipError_t train_pass(const TrainBatch& b, int d_in, int W, int D, int rows, float inv_n, const float* mean, const float* stdv,
                      const TrainWork& wk, const TrainState& st, int update, int cus, hipStream_t s) {
    const TrainData d{b.X, b.T, b.w, b.src_rows, d_in, b.rng, mean, stdv, b.seed, st.step};
    const bool small = rows <= kRows16 * cus * 256 / W;
    const dim3 grid(rows / (small ? 16 : 32)), block(4 * W);
#define ROWS_OF(WW, DD)                                                                                                \
    case WW * 8 + DD:                                                                                                  \
        if (small) hipLaunchKernelGGL((k_train_rows<WW, DD, 1>), grid, block, 0, s, d, st.theta, st.Wb, st.WbT, rows,  \
                                      inv_n, wk);                                                                      \
        else hipLaunchKernelGGL((k_train_rows<WW, DD, 2>), grid, block, 0, s, d, st.theta, st.Wb, st.WbT, rows, inv_n, \
                                wk);                                                                                   \
        break
    switch (W * 8 + D) {
        ROWS_OF(128, 2); ROWS_OF(128, 3); ROWS_OF(128, 4);
        ROWS_OF(256, 2); ROWS_OF(256, 3); ROWS_OF(256, 4);
        default: return hipErrorInvalidValue;
    }
#undef ROWS_OF
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const AdamArgs ad{st.theta, st.m1, st.m2, st.grad, st.step, st.lr, st.b1, st.b2, st.eps, update};
    const int side = W / 32, blocks = (D - 1) * side * side + (W / 16) * (d_in + D + 1) + 1;
    if (W == 256)
        hipLaunchKernelGGL(k_train_grads<256>, dim3(blocks), dim3(256), 0, s, D, d_in, rows, inv_n, wk, ad, st.Wb, st.WbT,
                           st.loss, st.step);
    else
        hipLaunchKernelGGL(k_train_grads<128>, dim3(blocks), dim3(256), 0, s, D, d_in, rows, inv_n, wk, ad, st.Wb, st.WbT,
                           st.loss, st.step);
    return hipGetLastError();
}

template <int W, int MT, int NT>
static hipError_t predict_of(const float* X, int64_t n, int d_in, int depth, const float* mean, const float* stdv,
                             const float* lo, const float* hi, int hull, const float* theta, const __bf16* Wb, float* Y,
                             uint8_t* in, hipStream_t s) {
    hipLaunchKernelGGL((k_predict<W, MT, NT>), dim3((unsigned)((n + 16 * MT - 1) / (16 * MT))), dim3(4 * W / NT), 0, s, X,
                       n, d_in, depth, mean, stdv, lo, hi, hull, theta, Wb, Y, in);
    return hipGetLastError();
}

template <int W>
static hipError_t predict_w(const float* X, int64_t n, int d_in, int depth, const float* mean, const float* stdv,
                            const float* lo, const float* hi, int hull, const float* theta, const __bf16* Wb, float* Y,
                            uint8_t* in, int cus, hipStream_t s) {
    // Few rows: the smallest tile, 16 rows, over as many CUs as there are, one unit tile per wave
    // (256 units: 16 waves).  More rows than 16 per CU: 32 rows per block of half the waves, two
    // blocks per CU, so that one's activations overlap the other's products (256 x 4, us per
    // launch: 5000 rows 16.1, against 25.7 with 64 rows per block; 32064 rows 53, against 59 with
    // 64 rows and 68 with 32 rows and all the waves).
    if (n <= kRows16 * cus) return predict_of<W, 1, 1>(X, n, d_in, depth, mean, stdv, lo, hi, hull, theta, Wb, Y, in, s);
    return predict_of<W, 2, 2>(X, n, d_in, depth, mean, stdv, lo, hi, hull, theta, Wb, Y, in, s);
}

hipError_t predict(const float* X, int64_t n, int d_in, int width, int depth, const float* mean, const float* stdv,
                   const float* lo, const float* hi, int hull, const float* theta, const __bf16* Wb, float* Y,
                   uint8_t* in, int cus, hipStream_t s) {
    switch (width) {
        case 64: return predict_w<64>(X, n, d_in, depth, mean, stdv, lo, hi, hull, theta, Wb, Y, in, cus, s);
        case 128: return predict_w<128>(X, n, d_in, depth, mean, stdv, lo, hi, hull, theta, Wb, Y, in, cus, s);
        case 192: return predict_w<192>(X, n, d_in, depth, mean, stdv, lo, hi, hull, theta, Wb, Y, in, cus, s);
        case 256: return predict_w<256>(X, n, d_in, depth, mean, stdv, lo, hi, hull, theta, Wb, Y, in, cus, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t first_forward(const float* Xn, int d_in, const float* W, const float* b, int width, int rows,
                         float* Z, __bf16* H, __bf16* HT, hipStream_t s) {
    hipLaunchKernelGGL(k_first_forward, grid1((int64_t)rows * width), dim3(kThreads), 0, s, Xn, d_in, W,
                       b, width, rows, Z, H, HT);
    return hipGetLastError();
}

hipError_t first_grad(const float* dZ, const float* Xn, int d_in, int width, int rows, float* dW,
                      float* db, hipStream_t s) {
    hipLaunchKernelGGL(k_first_grad, dim3(width), dim3(kThreads), 0, s, dZ, Xn, d_in, width, rows, dW, db);
    return hipGetLastError();
}

hipError_t colsum(const float* M, int width, int rows, float* out, hipStream_t s) {
    hipLaunchKernelGGL(k_colsum, dim3(width), dim3(kThreads), 0, s, M, width, rows, out);
    return hipGetLastError();
}

hipError_t output_layer(const float* Z, int width, int rows, const float* W, const float* b,
                        const float* T, const float* w, float inv_n, float* Y, float* dY,
                        float* rowloss, float* dZ, __bf16* dZb, __bf16* dZbT, hipStream_t s) {
    hipLaunchKernelGGL(k_output, dim3((rows + 3) / 4), dim3(kThreads), 0, s, Z, width, rows, W, b, T, w,
                       inv_n, Y, dY, rowloss, dZ, dZb, dZbT);
    return hipGetLastError();
}

hipError_t output_grad(const float* Z, int width, int rows, const float* dY, float* dW, float* db,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_output_grad, dim3(width + 1), dim3(kThreads), 0, s, Z, width, rows, dY, dW, db);
    return hipGetLastError();
}

hipError_t loss_sum(const float* rowloss, int rows, float inv_n, float* out, hipStream_t s) {
    hipLaunchKernelGGL(k_loss_sum, dim3(1), dim3(kThreads), 0, s, rowloss, rows, inv_n, out);
    return hipGetLastError();
}

hipError_t adam(float* theta, const float* grad, float* m1, float* m2, int64_t n, int64_t* step,
                const float* lr, float b1, float b2, float eps, hipStream_t s) {
    hipLaunchKernelGGL(k_adam, grid1(n), dim3(kThreads), 0, s, theta, grad, m1, m2, n, step, lr, b1, b2,
                       eps);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bump64, dim3(1), dim3(64), 0, s, step);
    return hipGetLastError();
}

hipError_t shadow(const float* W, int n_out, int n_in, __bf16* Wb, __bf16* WbT, hipStream_t s) {
    hipLaunchKernelGGL(k_shadow, grid1((int64_t)n_out * n_in), dim3(kThreads), 0, s, W, n_out, n_in, Wb,
                       WbT);
    return hipGetLastError();
}

hipError_t stats(const float* X, int d_in, int64_t n, float* mean, float* stdv, float* lo, float* hi,
                 hipStream_t s) {
    hipLaunchKernelGGL(k_stats, dim3(d_in), dim3(kThreads), 0, s, X, d_in, n, mean, stdv, lo, hi);
    return hipGetLastError();
}

hipError_t gather(const float* X, const float* T, const float* w, int64_t src_rows, int d_in, int rows,
                  const float* mean, const float* stdv, float* Xn, float* Tb, float* wb, int rng,
                  uint64_t seed, const int64_t* step, hipStream_t s) {
    hipLaunchKernelGGL(k_gather, grid1(rows), dim3(kThreads), 0, s, X, T, w, src_rows, d_in, rows, mean,
                       stdv, Xn, Tb, wb, rng, seed, step);
    return hipGetLastError();
}

hipError_t hull(const float* X, int d_in, int rows, const float* lo, const float* hi, uint8_t* in,
                hipStream_t s) {
    hipLaunchKernelGGL(k_hull, grid1(rows), dim3(kThreads), 0, s, X, d_in, rows, lo, hi, in);
    return hipGetLastError();
}

hipError_t normalise(const float* X, int64_t n, int d_in, int rows, const float* mean, const float* stdv,
                     float* Xn, hipStream_t s) {
    hipLaunchKernelGGL(k_normalise, grid1(rows), dim3(kThreads), 0, s, X, n, d_in, rows, mean, stdv, Xn);
    return hipGetLastError();
}

hipError_t fill_u8(uint8_t* p, int64_t n, uint8_t v, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_u8, grid1(n), dim3(kThreads), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t copy_u8(uint8_t* to, const uint8_t* from, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_u8, grid1(n), dim3(kThreads), 0, s, to, from, n);
    return hipGetLastError();
}

hipError_t init_params(float* theta, int64_t off, int n_out, int n_in, uint64_t seed, hipStream_t s) {
    hipLaunchKernelGGL(k_init_params, grid1((int64_t)n_out * n_in + n_out), dim3(kThreads), 0, s, theta,
                       off, n_out, n_in, seed);
    return hipGetLastError();
}

}  // namespace sur
}  // namespace scf
