// Refinement network kernels (gfx950): the training step (forward, loss,
// backward to the first layer in one kernel; the weight gradients with Adam
// on FP32 master weights in another), the fused inference, and the placement
// of the refined lattice.
//
// Network: g = [sin 2 pi B q, cos 2 pi B q] (B integer, 64 x 3), then four
// times h = GELU(W h + b) (128 -> 128), then s = W5 h + b5 (128 -> 3).  The
// loss is the mean over samples of |s - target|^2.  bf16 operands, FP32
// accumulation, FP32 master weights.
#include "tess_mlp.h"
#include "tess_tet.h"  // the connectivity table (kTet)

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

namespace tess {
namespace mlp {

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// D(16x16) += A(16x32) * B(32x16) on one wavefront.  Lane l supplies
// A[l % 16][8 (l / 16) + j] and B[8 (l / 16) + j][l % 16] (j = 0..7) and
// receives D[4 (l / 16) + i][l % 16] (i = 0..3).
__device__ inline floatx4 mma16(bf16x8 a, bf16x8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ inline float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// GELU(x) and its derivative (one erf for both).
__device__ inline void gelu_both(float x, float &h, float &g) {
    const float p = 1.0f + erff(x * 0.70710678118654752f);
    h = 0.5f * x * p;
    const float pdf = 0.39894228040143268f * __expf(-0.5f * x * x);
    g = 0.5f * p + x * pdf;
}

// SplitMix64 (Steele, Lea & Flood 2014): counter-based 64-bit mixer.
__host__ __device__ inline uint64_t splitmix64(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ inline double min_image(double d, double L) { return d - L * ceil(d / L - 0.5); }

// Sample j of minibatch `step`: a coarse vertex drawn with replacement by a
// counter hash, its q (unit torus) and target displacement s = (x - q L) / L,
// minimal image.
__device__ inline void gather_sample(const BatchSource &S, uint64_t step, int64_t j, float *__restrict__ q,
                                     float *__restrict__ target) {
    const int64_t n = (int64_t)S.d[0] * S.d[1] * S.d[2];
    const int64_t id = (int64_t)(splitmix64(S.seed ^ (step * 0x100000001B3ull + (uint64_t)j)) % (uint64_t)n);
    const int i = (int)(id % S.d[0]), jj = (int)((id / S.d[0]) % S.d[1]), k = (int)(id / ((int64_t)S.d[0] * S.d[1]));
    const double qu[3] = {(double)i / S.d[0], (double)jj / S.d[1], (double)k / S.d[2]};
    q[3 * j] = (float)qu[0];
    q[3 * j + 1] = (float)qu[1];
    q[3 * j + 2] = (float)qu[2];
    target[3 * j] = (float)(min_image((double)S.x[id] - qu[0] * S.L[0], S.L[0]) / S.L[0]);
    target[3 * j + 1] = (float)(min_image((double)S.y[id] - qu[1] * S.L[1], S.L[1]) / S.L[1]);
    target[3 * j + 2] = (float)(min_image((double)S.z[id] - qu[2] * S.L[2], S.L[2]) / S.L[2]);
}

__global__ void k_gather_batch(BatchSource S, uint64_t step, int64_t nb, float *__restrict__ q,
                               float *__restrict__ target) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < nb) gather_sample(S, step, j, q, target);
}

hipError_t launch_gather_batch(const BatchSource &S, uint64_t step, int64_t nb, float *q, float *target,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_gather_batch, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, S, step, nb, q, target);
    return hipGetLastError();
}

// ------------------------------------------------------- training step
// A training step is two launches: k_train_pass takes 32 samples per block
// through the features, the four layers forward, the output layer, the loss
// and back to the first layer, with every activation in LDS and registers;
// k_train_grads sums the weight gradients and updates the parameters.  In
// between only the activations H and the errors dZ cross memory, transposed
// (feature-major, `ld` samples per feature), which is the layout in which
// the gradient's contraction over the samples reads both operands in 16-byte
// pieces.  (A launch per layer and operation, 25 a step, took 430 us a step
// at 8192 samples: each kernel was shorter than its launch and start-up,
// the gradients went through 34 MB of partial sums written and read back,
// and the output layer's backward read its FP32 pre-activations row by row.)
//
// k_train_pass: wavefront w owns output columns 16 w .. 16 w + 15 of every
// layer for both 16-row tiles, so that its weights are 4 KB per layer, read
// once, a layer ahead, straight into the MFMA's B operand; GELU' of its
// pre-activations stays in its registers for the way back.
constexpr int kTrainRows = 32, kTrainThreads = 512;

__global__ void __launch_bounds__(kTrainThreads) k_train_pass(TrainNet T, int64_t n, int64_t ld) {
    constexpr int LDA = kWidth + 8;  // padded row (bf16 elements)
    __shared__ bf16 sA[2][kTrainRows * LDA];
    __shared__ float sW5[3 * kWidth + 3];
    __shared__ float sB[3 * kFreq];
    __shared__ float sQ[3 * kTrainRows], sE[3 * kTrainRows];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lq = lane >> 4, lk = 8 * lq;
    const int64_t row0 = (int64_t)blockIdx.x * kTrainRows;
    const int col = 16 * wave + lr;
    bf16x8 w[4];  // this wavefront's columns of the next product's matrix
    auto load_w = [&](const bf16 *M) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) w[ks] = *(const bf16x8 *)&M[col * kWidth + ks * 32 + lk];
    };
    load_w(T.Wb);
    for (int e = threadIdx.x; e < 3 * kWidth; e += kTrainThreads) sW5[e] = (float)(bf16)T.master[kOffW5 + e];
    if (threadIdx.x < 3) sW5[3 * kWidth + threadIdx.x] = T.master[kOffB5 + threadIdx.x];
    if (threadIdx.x < 3 * kFreq) sB[threadIdx.x] = T.B[threadIdx.x];
    if (threadIdx.x < 3 * kTrainRows) {
        const int64_t e = 3 * row0 + threadIdx.x;
        sQ[threadIdx.x] = e < 3 * n ? T.q[e] : 0.f;
    }
    __syncthreads();
    // features: sin(2 pi B_f . q) and cos(...) (B is integer, so sinpi and
    // cospi of 2 B.q reduce exactly for dyadic q)
    {
        const int f = threadIdx.x & (kFreq - 1);
        for (int r = threadIdx.x >> 6; r < kTrainRows; r += kTrainThreads / 64) {
            const float t = 2.0f * (sB[3 * f] * sQ[3 * r] + sB[3 * f + 1] * sQ[3 * r + 1] + sB[3 * f + 2] * sQ[3 * r + 2]);
            sA[0][r * LDA + f] = (bf16)sinpif(t);
            sA[0][r * LDA + kFreq + f] = (bf16)cospif(t);
        }
    }
    __syncthreads();
    {  // transposed copy: 8 samples of one feature per thread
        const int c = threadIdx.x >> 2, r8 = 8 * (threadIdx.x & 3);
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = row0 + r8 + j < n ? sA[0][(r8 + j) * LDA + c] : (bf16)0.0f;
        *(bf16x8 *)&T.act[(int64_t)c * ld + row0 + r8] = v;
    }
    // one product of the 32 rows in sA[cur] with this wavefront's columns
    auto product = [&](int cur, floatx4 acc[2]) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            acc[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16x8 a = *(const bf16x8 *)&sA[cur][(rt * 16 + lr) * LDA + ks * 32 + lk];
                acc[rt] = mma16(a, w[ks], acc[rt]);
            }
        }
    };
    // the values v of this lane's rows 16 rt + 4 lq + i: to LDS for the next
    // product and, transposed, to memory (zeros past the last sample)
    auto put = [&](int nxt, const float v[2][4], bf16 *__restrict__ out) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            bf16x4 p;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * rt + 4 * lq + i;
                p[i] = (bf16)v[rt][i];
                sA[nxt][r * LDA + col] = p[i];
                if (row0 + r >= n) p[i] = (bf16)0.0f;
            }
            *(bf16x4 *)&out[(int64_t)col * ld + row0 + 16 * rt + 4 * lq] = p;
        }
    };
    const int64_t plane = (int64_t)kWidth * ld;
    float G[kDepth][2][4];
#pragma unroll
    for (int l = 0; l < kDepth; ++l) {
        floatx4 acc[2];
        product(l & 1, acc);
        load_w(l + 1 < kDepth ? T.Wb + (size_t)(l + 1) * kWidth * kWidth : T.WTb + (size_t)l * kWidth * kWidth);
        const float bias = T.master[param_offset_b(l) + col];
        float v[2][4];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int i = 0; i < 4; ++i) gelu_both(acc[rt][i] + bias, v[rt][i], G[l][rt][i]);
        put(1 - (l & 1), v, T.act + (l + 1) * plane);
        __syncthreads();
    }
    static_assert(kDepth % 2 == 0, "the last activations are in buffer 0");
    // output layer, a thread per (sample, component), and the error
    if (threadIdx.x < 3 * kTrainRows) {
        const int r = threadIdx.x / 3, c = threadIdx.x % 3;
        float a = 0.f;
        for (int i = 0; i < kWidth; i += 8) {
            const bf16x8 h = *(const bf16x8 *)&sA[0][r * LDA + i];
#pragma unroll
            for (int j = 0; j < 8; ++j) a += (float)h[j] * sW5[c * kWidth + i + j];
        }
        const float p = a + sW5[3 * kWidth + c];
        const int64_t e = 3 * row0 + threadIdx.x;
        float err = 0.f;
        if (e < 3 * n) {
            T.pred[e] = p;
            err = p - T.target[e];
        }
        sE[threadIdx.x] = err;
    }
    __syncthreads();
    const float sc = 2.0f / (float)n;
    if (threadIdx.x < kTrainRows) {
        const float e0 = sE[3 * threadIdx.x], e1 = sE[3 * threadIdx.x + 1], e2 = sE[3 * threadIdx.x + 2];
        T.dout[3 * ld + row0 + threadIdx.x] = e0 * e0 + e1 * e1 + e2 * e2;
    }
    if (threadIdx.x < 3 * kTrainRows) {
        const int c = threadIdx.x / kTrainRows, r = threadIdx.x % kTrainRows;
        T.dout[c * ld + row0 + r] = sc * sE[3 * r + c];
    }
    {
        float v[2][4];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * rt + 4 * lq + i;
                const float d0 = sc * sE[3 * r], d1 = sc * sE[3 * r + 1], d2 = sc * sE[3 * r + 2];
                const float g = d0 * sW5[col] + d1 * sW5[kWidth + col] + d2 * sW5[2 * kWidth + col];
                v[rt][i] = g * G[kDepth - 1][rt][i];
            }
        put(1, v, T.err + (kDepth - 1) * plane);
    }
    __syncthreads();
#pragma unroll
    for (int l = kDepth - 1; l > 0; --l) {
        floatx4 acc[2];
        product(l & 1, acc);
        if (l > 1) load_w(T.WTb + (size_t)(l - 1) * kWidth * kWidth);
        float v[2][4];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[rt][i] = acc[rt][i] * G[l - 1][rt][i];
        put(1 - (l & 1), v, T.err + (l - 1) * plane);
        __syncthreads();
    }
}

hipError_t launch_train_pass(const TrainNet &T, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_train_pass, dim3((unsigned)(train_rows(n) / kTrainRows)), dim3(kTrainThreads), 0, s, T, n,
                       train_rows(n));
    return hipGetLastError();
}

// Weight gradients and (ADAM) the parameter update, the transposed bf16
// copies and the next minibatch.  Sums keep one fixed order: within a slice
// of kSlice samples by the MFMA (hidden weights) or one sample after
// another (biases; the output layer takes slices of kOutSlice), then slice
// after slice, in FP32.  Blocks:
//   0 .. 255   one 16 x 16 tile of a hidden layer's weights each: the
//              wavefronts take slices in turn, the slices' sums meet in LDS
//              and are added there in slice order (through memory they would
//              be 34 MB a step at 8192 samples).  A layer's tiles sit on two
//              of the eight XCDs (blocks go round the XCDs), whose L2 then
//              holds that layer's 4 MB of operands at 8192 samples;
//   256 .. 287 16 biases of a hidden layer each (in the tiles' blocks their
//              serial sums held up a row of tiles: 25 us against 19);
//   288 .. 319 4 columns of the output layer's weights each;
//   320        the output biases and (on request) the loss;
//   321 ..     the next minibatch, 512 samples each.
// The blocks read the activations and errors and write their own
// parameters; none reads what another writes.
constexpr int kGradThreads = 512, kGradChunk = 64, kOutSlice = 256;
constexpr int kGradTiles = kDepth * 64, kGradBias = kGradTiles + kDepth * 8;
constexpr int kGradOutCols = 4;  // columns of the output layer per block
constexpr int kGradOut = kGradBias + kWidth / kGradOutCols, kGradRest = kGradOut + 1;

template <bool ADAM>
__global__ void __launch_bounds__(kGradThreads) k_train_grads(TrainNet T, int64_t n, int64_t ld, AdamStep A,
                                                              float *__restrict__ grad, float *__restrict__ loss,
                                                              BatchSource S, uint64_t next) {
    constexpr int kWaves = kGradThreads / 64;
    constexpr int LP = 256;  // sums of one slice
    __shared__ float part[kGradChunk * LP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lq = lane >> 4, lk = 8 * lq;
    const int64_t plane = (int64_t)kWidth * ld;
    // a parameter's gradient g is complete: the update, or the gradient itself
    auto finish = [&](int64_t e, float g) -> float {
        if constexpr (ADAM) {
            const float mi = A.b1 * T.m[e] + A.a1 * g;
            const float vi = A.b2 * T.v[e] + A.a2 * g * g;
            T.m[e] = mi;
            T.v[e] = vi;
            float w = T.master[e];
            w -= A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + A.eps);
            T.master[e] = w;
            return w;
        } else {
            grad[e] = g;
            return 0.f;
        }
    };
    if (blockIdx.x < kGradTiles) {
        const int l = (int)(blockIdx.x & 7u) >> 1, tile = (int)(blockIdx.x >> 3) * 2 + (int)(blockIdx.x & 1u);
        const int to = tile >> 3, ti = tile & 7;
        const bf16 *dz = T.err + l * plane + (int64_t)(16 * to) * ld;
        const bf16 *hh = T.act + l * plane + (int64_t)(16 * ti) * ld;
        const int64_t slices = (n + kSlice - 1) / kSlice;
        float sum = 0.f;  // thread t < 256: element t
        for (int64_t k0 = 0; k0 < slices; k0 += kGradChunk) {
            const int nk = (int)(slices - k0 < kGradChunk ? slices - k0 : kGradChunk);
            // four slices' operands in flight per wavefront (one at a time
            // waits for memory 16 times)
            for (int kb = wave; kb < nk; kb += 4 * kWaves) {
                bf16x8 a[4][kSlice / 32], b[4][kSlice / 32];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = kb + u * kWaves < nk ? kb + u * kWaves : kb;
                    const int64_t at = (int64_t)lr * ld + (k0 + k) * kSlice + lk;
#pragma unroll
                    for (int ks = 0; ks < kSlice / 32; ++ks) {
                        a[u][ks] = *(const bf16x8 *)&dz[at + 32 * ks];
                        b[u][ks] = *(const bf16x8 *)&hh[at + 32 * ks];
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = kb + u * kWaves;
                    if (k >= nk) break;
                    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < kSlice / 32; ++ks) acc = mma16(a[u][ks], b[u][ks], acc);
#pragma unroll
                    for (int i = 0; i < 4; ++i) part[k * LP + (4 * lq + i) * 16 + lr] = acc[i];
                }
            }
            __syncthreads();
            if (threadIdx.x < 256)
#pragma unroll 8
                for (int k = 0; k < nk; ++k) sum += part[k * LP + threadIdx.x];
            __syncthreads();
        }
        if (threadIdx.x < 256) {
            const int r = 16 * to + (threadIdx.x >> 4), c = 16 * ti + (threadIdx.x & 15);
            const float w = finish(param_offset_W(l) + r * kWidth + c, sum);
            if constexpr (ADAM) {
                T.Wb[(size_t)l * kWidth * kWidth + r * kWidth + c] = (bf16)w;
                T.WTb[(size_t)l * kWidth * kWidth + c * kWidth + r] = (bf16)w;
            }
        }
        return;
    }
    if (blockIdx.x < kGradBias) {
        // 16 biases of a hidden layer
        const int l = (int)(blockIdx.x - kGradTiles) >> 3, o0 = 16 * ((int)(blockIdx.x - kGradTiles) & 7);
        const bf16 *dz = T.err + l * plane + (int64_t)o0 * ld;
        const int64_t slices = (n + kSlice - 1) / kSlice;
        float sum = 0.f;
        for (int64_t k0 = 0; k0 < slices; k0 += kGradChunk) {
            const int nk = (int)(slices - k0 < kGradChunk ? slices - k0 : kGradChunk);
            for (int c = threadIdx.x; c < 16 * nk; c += kGradThreads) {
                const int o = c / nk, k = c - o * nk;
                bf16x8 v[kSlice / 8];
#pragma unroll
                for (int j = 0; j < kSlice / 8; ++j)
                    v[j] = *(const bf16x8 *)&dz[(int64_t)o * ld + (k0 + k) * kSlice + 8 * j];
                float s = 0.f;
#pragma unroll
                for (int j = 0; j < kSlice; ++j) s += (float)v[j >> 3][j & 7];
                part[k * LP + o] = s;
            }
            __syncthreads();
            if (threadIdx.x < 16)
#pragma unroll 8
                for (int k = 0; k < nk; ++k) sum += part[k * LP + threadIdx.x];
            __syncthreads();
        }
        if (threadIdx.x < 16) finish(param_offset_b(l) + o0 + threadIdx.x, sum);
        return;
    }
    const int64_t oslices = (n + kOutSlice - 1) / kOutSlice;
    if (blockIdx.x < kGradOut) {
        // dW5[c][i] = sum of d[c] H4[i] over the samples
        constexpr int NC = kGradOutCols;
        const int i0 = NC * (int)(blockIdx.x - kGradBias);
        const bf16 *h4 = T.act + kDepth * plane;
        float sum = 0.f;
        for (int64_t k0 = 0; k0 < oslices; k0 += kGradChunk) {
            const int nk = (int)(oslices - k0 < kGradChunk ? oslices - k0 : kGradChunk);
            for (int t = threadIdx.x; t < 3 * NC * nk; t += kGradThreads) {
                const int e = t % (3 * NC), k = t / (3 * NC), c = e / NC;
                const int64_t r0 = (k0 + k) * kOutSlice;
                const bf16 *hp = h4 + (int64_t)(i0 + e % NC) * ld;
                const float *dp = T.dout + c * ld;
                float s = 0.f;
                // 32 samples' loads together (ld is a multiple of 64, zeros from n on)
                for (int r = 0; r < kOutSlice && r0 + r < ld; r += 32) {
                    bf16x8 v[4];
                    floatx4 d[8];
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = *(const bf16x8 *)&hp[r0 + r + 8 * j];
#pragma unroll
                    for (int j = 0; j < 8; ++j) d[j] = *(const floatx4 *)&dp[r0 + r + 4 * j];
#pragma unroll
                    for (int j = 0; j < 32; ++j) s += d[j >> 2][j & 3] * (float)v[j >> 3][j & 7];
                }
                part[k * LP + e] = s;
            }
            __syncthreads();
            if (threadIdx.x < 3 * NC)
#pragma unroll 8
                for (int k = 0; k < nk; ++k) sum += part[k * LP + threadIdx.x];
            __syncthreads();
        }
        if (threadIdx.x < 3 * NC) finish(kOffW5 + threadIdx.x / NC * kWidth + i0 + threadIdx.x % NC, sum);
        return;
    }
    if (blockIdx.x == kGradOut) {
        // sums of the rows of dout: the three output biases, then the loss
        const int rows = loss ? 4 : 3;
        float sum = 0.f;
        for (int64_t k0 = 0; k0 < oslices; k0 += kGradChunk) {
            const int nk = (int)(oslices - k0 < kGradChunk ? oslices - k0 : kGradChunk);
            for (int t = threadIdx.x; t < rows * nk; t += kGradThreads) {
                const int c = t % rows, k = t / rows;
                const int64_t r0 = (k0 + k) * kOutSlice;
                float s = 0.f;
                for (int r = 0; r < kOutSlice && r0 + r < ld; r += 64) {
                    floatx4 v[16];
#pragma unroll
                    for (int j = 0; j < 16; ++j) v[j] = *(const floatx4 *)&T.dout[c * ld + r0 + r + 4 * j];
#pragma unroll
                    for (int j = 0; j < 64; ++j) s += v[j >> 2][j & 3];
                }
                part[k * LP + c] = s;
            }
            __syncthreads();
            if (threadIdx.x < rows)
                for (int k = 0; k < nk; ++k) sum += part[k * LP + threadIdx.x];
            __syncthreads();
        }
        if (threadIdx.x < 3) finish(kOffB5 + threadIdx.x, sum);
        else if (threadIdx.x == 3 && loss) *loss = sum;
        return;
    }
    if constexpr (ADAM) {
        const int64_t j = (int64_t)(blockIdx.x - kGradRest) * kGradThreads + threadIdx.x;
        if (j < n) gather_sample(S, next, j, T.q, T.target);
    }
}

hipError_t launch_train_grads(const TrainNet &T, int64_t n, float *grad, float *loss, hipStream_t s) {
    hipLaunchKernelGGL(k_train_grads<false>, dim3(kGradRest), dim3(kGradThreads), 0, s, T, n, train_rows(n), AdamStep{},
                       grad, loss, BatchSource{}, (uint64_t)0);
    return hipGetLastError();
}

hipError_t launch_train_update(const TrainNet &T, int64_t n, const AdamStep &A, float *loss, const BatchSource &S,
                               uint64_t next, hipStream_t s) {
    const int64_t more = next ? (n + kGradThreads - 1) / kGradThreads : 0;
    hipLaunchKernelGGL(k_train_grads<true>, dim3((unsigned)(kGradRest + more)), dim3(kGradThreads), 0, s, T, n,
                       train_rows(n), A, (float *)nullptr, loss, S, next);
    return hipGetLastError();
}

// ----------------------------------------------------------------- Adam
// a1 = 1 - b1, a2 = 1 - b2 and the bias corrections c = 1 - b^t come from
// the host in FP64: in FP32 each difference cancels several digits (with
// b2 = 0.999, 1 - b2^t at small t keeps only about 4 of them)
AdamStep adam_step(double lr, double b1, double b2, double eps, int t) {
    const double c1 = 1.0 - std::pow(b1, (double)t), c2 = 1.0 - std::pow(b2, (double)t);
    return AdamStep{(float)lr, (float)b1, (float)(1.0 - b1), (float)b2, (float)(1.0 - b2), (float)eps, (float)c1,
                    (float)c2};
}

// In-place Adam on FP32 master parameters (bias-corrected, step t >= 1).
__global__ void k_adam(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ g, int64_t count, AdamStep A) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    const float gi = g[e];
    const float mi = A.b1 * m[e] + A.a1 * gi;
    const float vi = A.b2 * v[e] + A.a2 * gi * gi;
    m[e] = mi;
    v[e] = vi;
    w[e] -= A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + A.eps);
}

hipError_t launch_adam(float *w, float *m, float *v, const float *g, int64_t count, const AdamStep &A,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, w, m, v, g, count, A);
    return hipGetLastError();
}

// ------------------------------------------------------ fused inference
// The whole forward pass of one 16-sample tile on one wavefront, for
// inference: the features, the four hidden layers and the output layer stay
// in registers.  Each layer is computed transposed, D = W H^T (the weights
// as the MFMA's A operand, the activations as its B operand), so that after
// a layer the lane holding sample r = l % 16 has outputs o = 16 ot + 4 q + i
// (q = l / 16, i < 4, ot < 8): exactly the B operand of the next layer if
// that layer takes its input columns in the order k = 32 ks + 8 q + j <->
// input feature perm(k) = 16 (2 ks + j / 4) + 4 q + j % 4.  The weights are
// staged in LDS in that order, one 16-byte A fragment per lane per (layer,
// ot, ks); the first layer takes the features in their natural order, which
// the lanes compute for themselves.
//
// What bounds it is the activations' vector instructions (128 GELUs a lane
// and tile; the MFMAs are a seventh of that, the fragments' LDS reads a
// third).  They come in dependent chains behind branches, so it takes the
// four wavefronts per SIMD that 128 registers admit to fill them: 2^20
// points 485 us with two per SIMD and a bias read per value, 417 us with
// four biases per read, 343 us with four wavefronts.  (Two tiles per
// wavefront, which halves the LDS reads, at two wavefronts: 394 us.)
constexpr int kInferWaves = 16;           // 1024 threads; the staged weights admit one block per CU
constexpr int kFragsHidden = kDepth * 8 * 4 * 64;  // 16-byte fragments of the four hidden layers
constexpr int kFragsOut = 4 * 64;         // of the output layer (3 of its 16 rows are real)

__device__ __host__ inline int infer_perm(int k) {
    const int ks = k >> 5, q = (k >> 3) & 3, j = k & 7;
    return 16 * (2 * ks + (j >> 2)) + 4 * q + (j & 3);
}

__global__ void __launch_bounds__(64 * kInferWaves) k_mlp_infer(const float *__restrict__ q, int64_t n,
                                                                const float *__restrict__ B,
                                                                const float *__restrict__ master,
                                                                float *__restrict__ pred) {
    extern __shared__ bf16x8 sFrag[];                 // hidden, then output fragments
    __shared__ __align__(16) float sBias[kDepth * kWidth + 4];
    __shared__ float sB[3 * kFreq];
    // stage: fragment f of (layer, ot, ks, lane) holds W[o][perm or natural k .. +7]:
    // two runs of four columns (16-byte loads: rows and layers start at
    // multiples of four parameters of an allocation)
#pragma unroll 3
    for (int f = threadIdx.x; f < kFragsHidden + kFragsOut; f += blockDim.x) {
        const int lane = f & 63, ks = (f >> 6) & 3;
        const bool out = f >= kFragsHidden;
        const int ot = out ? 0 : (f >> 8) & 7, l = out ? kDepth : f >> 11;
        const int o = 16 * ot + (lane & 15);
        const int lq = lane >> 4;
        const int k0 = l == 0 ? 32 * ks + 8 * lq : infer_perm(32 * ks + 8 * lq);
        const int k1 = l == 0 ? k0 + 4 : infer_perm(32 * ks + 8 * lq + 4);
        const float *row = master + param_offset_W(l) + (int64_t)o * kWidth;  // (the output layer's follow the hidden ones')
        floatx4 w0 = {0.f, 0.f, 0.f, 0.f}, w1 = w0;
        if (!out || o < 3) {
            w0 = *(const floatx4 *)&row[k0];
            w1 = *(const floatx4 *)&row[k1];
        }
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = (bf16)w0[j];
            v[4 + j] = (bf16)w1[j];
        }
        sFrag[f] = v;
    }
    for (int e = threadIdx.x; e < kDepth * kWidth; e += blockDim.x)
        sBias[e] = master[param_offset_b(e / kWidth) + e % kWidth];
    if (threadIdx.x < 3) sBias[kDepth * kWidth + threadIdx.x] = master[kOffB5 + threadIdx.x];
    for (int e = threadIdx.x; e < 3 * kFreq; e += blockDim.x) sB[e] = B[e];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lq = lane >> 4, lr = lane & 15;
    const int64_t ntile = (n + 15) / 16;
    // (neighbouring tiles on neighbouring CUs: a small call has a tile on each)
    for (int64_t tile = (int64_t)wave * gridDim.x + blockIdx.x; tile < ntile;
         tile += (int64_t)gridDim.x * kInferWaves) {
        const int64_t row = tile * 16 + lr;
        const bool live = row < n;
        // features of sample `row`, k = 32 ks + 8 q + j (natural order: sin
        // of frequency k for k < 64, cos of frequency k - 64 above)
        // (columns 64 apart are the sine and cosine of one frequency: k and
        // k + 64 sit in blocks ks and ks + 2 of the same lane)
        bf16x8 h[4];
        {
            int own = 0;  // (opaque: the frequencies are read again for each tile, not kept in 48 registers)
            asm volatile("" : "+v"(own));
            const float *fB = sB + own;
            const float q0 = live ? q[3 * row] : 0.f, q1 = live ? q[3 * row + 1] : 0.f,
                        q2 = live ? q[3 * row + 2] : 0.f;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int f = 32 * ks + 8 * lq + j;
                    const float t = 2.0f * (fB[3 * f] * q0 + fB[3 * f + 1] * q1 + fB[3 * f + 2] * q2);
                    float sv, cv;
                    sincospif(t, &sv, &cv);
                    h[ks][j] = (bf16)sv;
                    h[ks + 2][j] = (bf16)cv;
                }
        }
#pragma unroll 1
        for (int l = 0; l < kDepth; ++l) {
            floatx4 acc[8];
#pragma unroll
            for (int ot = 0; ot < 8; ++ot) {
                acc[ot] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc[ot] = mma16(sFrag[((l * 8 + ot) * 4 + ks) * 64 + lane], h[ks], acc[ot]);
            }
            // bias, GELU, bf16: the next layer's operand (outputs 16 ot + 4 q + i
            // of this lane's sample, in the next layer's column order)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                floatx4 bias[2];
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    bias[e] = *(const floatx4 *)&sBias[l * kWidth + 16 * (2 * ks + e) + 4 * lq];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    h[ks][j] = (bf16)gelu(acc[2 * ks + (j >> 2)][j & 3] + bias[j >> 2][j & 3]);
            }
        }
        floatx4 out = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) out = mma16(sFrag[kFragsHidden + ks * 64 + lane], h[ks], out);
        // lanes 0..15 hold outputs 0..3 of their sample (3 are real)
        if (lq == 0 && live) {
            pred[3 * row] = out[0] + sBias[kDepth * kWidth];
            pred[3 * row + 1] = out[1] + sBias[kDepth * kWidth + 1];
            pred[3 * row + 2] = out[2] + sBias[kDepth * kWidth + 2];
        }
    }
}

hipError_t launch_mlp_infer(const float *q, int64_t n, const float *B, const float *master, float *pred,
                            hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int64_t tiles = (n + 15) / 16;
    const int blocks = (int)std::min<int64_t>(tiles, (int64_t)cus);
    const size_t lds = sizeof(bf16x8) * (size_t)(kFragsHidden + kFragsOut);
    hipLaunchKernelGGL(k_mlp_infer, dim3((unsigned)blocks), dim3(64 * kInferWaves), lds, s, q, n, B, master, pred);
    return hipGetLastError();
}

// bf16 copies of the four hidden weight matrices, row-major and transposed.
__global__ void k_cast_weights(const float *__restrict__ master, bf16 *__restrict__ Wb,
                               bf16 *__restrict__ WTb) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= kDepth * kWidth * kWidth) return;
    const int l = e / (kWidth * kWidth), r = (e / kWidth) % kWidth, c = e % kWidth;
    const float w = master[param_offset_W(l) + r * kWidth + c];
    Wb[e] = (bf16)w;
    WTb[l * kWidth * kWidth + c * kWidth + r] = (bf16)w;
}

hipError_t launch_cast_weights(const float *master, bf16 *Wb, bf16 *WTb, hipStream_t s) {
    const int total = kDepth * kWidth * kWidth;
    hipLaunchKernelGGL(k_cast_weights, dim3((total + 255) / 256), dim3(256), 0, s, master, Wb, WTb);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace tess

namespace tess {
namespace mlp {

// ------------------------------------------------------ refinement glue
// Unit-torus coordinates of fine vertices first .. first + n - 1 (id order).
__global__ void k_fine_q(int64_t first, int64_t n, int f0, int f1, int f2, float *__restrict__ q) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int64_t id = first + j;
    q[3 * j] = (float)((double)(id % f0) / f0);
    q[3 * j + 1] = (float)((double)((id / f0) % f1) / f1);
    q[3 * j + 2] = (float)((double)(id / ((int64_t)f0 * f1)) / f2);
}

hipError_t launch_fine_q(int64_t first, int64_t n, const int fdims[3], float *q, hipStream_t s) {
    hipLaunchKernelGGL(k_fine_q, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, first, n, fdims[0],
                       fdims[1], fdims[2], q);
    return hipGetLastError();
}

__device__ inline float wrap_f32(double v, double L) {
    double w = v - L * floor(v / L);
    float f = (float)w;
    if (f >= (float)L) f -= (float)L;
    if (f < 0.f) f = 0.f;
    return f;
}

// Fine positions from the network: coarse vertices keep their data, the
// others get q L + s(q) L, wrapped into the box.
__global__ void k_place_mlp(const float *__restrict__ cx, const float *__restrict__ cy,
                            const float *__restrict__ cz, int d0, int d1, int r, int64_t first,
                            int64_t n, const float *__restrict__ q, const float *__restrict__ pred,
                            double L0, double L1, double L2, int f0, int f1, float *__restrict__ fx,
                            float *__restrict__ fy, float *__restrict__ fz) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int64_t id = first + j;
    const int I = (int)(id % f0), J = (int)((id / f0) % f1), K = (int)(id / ((int64_t)f0 * f1));
    if (I % r == 0 && J % r == 0 && K % r == 0) {
        const int64_t c = (int64_t)(I / r) + (int64_t)d0 * ((J / r) + (int64_t)d1 * (K / r));
        fx[id] = cx[c];
        fy[id] = cy[c];
        fz[id] = cz[c];
        return;
    }
    fx[id] = wrap_f32(((double)q[3 * j] + (double)pred[3 * j]) * L0, L0);
    fy[id] = wrap_f32(((double)q[3 * j + 1] + (double)pred[3 * j + 1]) * L1, L1);
    fz[id] = wrap_f32(((double)q[3 * j + 2] + (double)pred[3 * j + 2]) * L2, L2);
}

hipError_t launch_place_mlp(const float *cx, const float *cy, const float *cz, const int cdims[3], int r,
                            int64_t first, int64_t n, const float *q, const float *pred,
                            const double box[3], const int fdims[3], float *fx, float *fy, float *fz,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_place_mlp, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cx, cy, cz,
                       cdims[0], cdims[1], r, first, n, q, pred, box[0], box[1], box[2], fdims[0], fdims[1],
                       fx, fy, fz);
    return hipGetLastError();
}

// The tetrahedron of the unit cube's six-tetrahedron table (corner n = a +
// 2b + 4c at offset (a, b, c)) that contains point p, and p's barycentric
// coordinates in it (Cramer's rule); -1 if none does (not reached for points
// of the unit cube, which the six tetrahedra tile).
__device__ inline int unit_cube_tet(const double p[3], double lam[4]) {
    for (int t = 0; t < 6; ++t) {
        double R[4][3];
        for (int m = 0; m < 4; ++m) {
            const int c = kTet[t][m];
            R[m][0] = c & 1; R[m][1] = (c >> 1) & 1; R[m][2] = (c >> 2) & 1;
        }
        double M[3][3], rhs[3];
        for (int a = 0; a < 3; ++a) {
            for (int m = 0; m < 3; ++m) M[a][m] = R[m + 1][a] - R[0][a];
            rhs[a] = p[a] - R[0][a];
        }
        const double det = M[0][0] * (M[1][1] * M[2][2] - M[1][2] * M[2][1]) -
                           M[0][1] * (M[1][0] * M[2][2] - M[1][2] * M[2][0]) +
                           M[0][2] * (M[1][0] * M[2][1] - M[1][1] * M[2][0]);
        for (int m = 0; m < 3; ++m) {
            double T[3][3];
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) T[a][b] = (b == m) ? rhs[a] : M[a][b];
            lam[m + 1] = (T[0][0] * (T[1][1] * T[2][2] - T[1][2] * T[2][1]) -
                          T[0][1] * (T[1][0] * T[2][2] - T[1][2] * T[2][0]) +
                          T[0][2] * (T[1][0] * T[2][1] - T[1][1] * T[2][0])) / det;
        }
        lam[0] = 1.0 - lam[1] - lam[2] - lam[3];
        if (lam[0] < -1e-12 || lam[1] < -1e-12 || lam[2] < -1e-12 || lam[3] < -1e-12) continue;
        return t;
    }
    return -1;
}

__device__ inline int cube_corner(int t, int m) { return kTet[t][m]; }

// Fine positions by the affine map of the coarse tetrahedron that contains
// the vertex's Lagrangian point.
__global__ void k_place_linear(const float *__restrict__ cx, const float *__restrict__ cy,
                               const float *__restrict__ cz, int d0, int d1, int d2, int r,
                               double L0, double L1, double L2, int64_t nfine,
                               float *__restrict__ fx, float *__restrict__ fy, float *__restrict__ fz) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= nfine) return;
    const int f0 = d0 * r, f1 = d1 * r;
    const int I = (int)(id % f0), J = (int)((id / f0) % f1), K = (int)(id / ((int64_t)f0 * f1));
    const int i = I / r, j = J / r, k = K / r;
    const double p[3] = {(double)(I % r) / r, (double)(J % r) / r, (double)(K % r) / r};
    const double L[3] = {L0, L1, L2};
    // unwrapped corners of the coarse cube (periodic image nearest corner 0)
    double X[8][3];
    for (int c = 0; c < 8; ++c) {
        int ii = i + (c & 1), jj = j + ((c >> 1) & 1), kk = k + ((c >> 2) & 1);
        if (ii == d0) ii = 0;
        if (jj == d1) jj = 0;
        if (kk == d2) kk = 0;
        const int64_t cid = ii + (int64_t)d0 * (jj + (int64_t)d1 * kk);
        const double v[3] = {(double)cx[cid], (double)cy[cid], (double)cz[cid]};
        for (int a = 0; a < 3; ++a) {
            if (c == 0) {
                X[0][a] = v[a];
            } else {
                double e = v[a] - X[0][a];
                e -= L[a] * ceil(e / L[a] - 0.5);
                X[c][a] = X[0][a] + e;
            }
        }
    }
    double lam[4];
    const int t = unit_cube_tet(p, lam);
    double out[3] = {X[0][0], X[0][1], X[0][2]};
    if (t >= 0) {
        out[0] = out[1] = out[2] = 0.0;
        for (int m = 0; m < 4; ++m)
            for (int a = 0; a < 3; ++a) out[a] += lam[m] * X[cube_corner(t, m)][a];
    }
    fx[id] = wrap_f32(out[0], L0);
    fy[id] = wrap_f32(out[1], L1);
    fz[id] = wrap_f32(out[2], L2);
}

hipError_t launch_place_linear(const float *cx, const float *cy, const float *cz, const int cdims[3], int r,
                               const double box[3], float *fx, float *fy, float *fz, hipStream_t s) {
    const int64_t nfine = (int64_t)cdims[0] * cdims[1] * cdims[2] * r * r * r;
    hipLaunchKernelGGL(k_place_linear, dim3((unsigned)((nfine + 255) / 256)), dim3(256), 0, s, cx, cy, cz,
                       cdims[0], cdims[1], cdims[2], r, box[0], box[1], box[2], nfine, fx, fy, fz);
    return hipGetLastError();
}

// Residual of the network at coarse tracers first .. first+n-1 (q and pred
// of those tracers): x - (q + s(q)) L, as the periodic image in (-L/2, L/2].
__global__ void k_coarse_residual(const float *__restrict__ cx, const float *__restrict__ cy,
                                  const float *__restrict__ cz, int64_t first, int64_t n,
                                  const float *__restrict__ q, const float *__restrict__ pred, double L0,
                                  double L1, double L2, float *__restrict__ rx, float *__restrict__ ry,
                                  float *__restrict__ rz) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int64_t id = first + j;
    const double x[3] = {(double)cx[id], (double)cy[id], (double)cz[id]};
    const double L[3] = {L0, L1, L2};
    float *out[3] = {rx, ry, rz};
    for (int a = 0; a < 3; ++a) {
        double d = x[a] - ((double)q[3 * j + a] + (double)pred[3 * j + a]) * L[a];
        d -= L[a] * ceil(d / L[a] - 0.5);
        out[a][id] = (float)d;
    }
}

hipError_t launch_coarse_residual(const float *cx, const float *cy, const float *cz, int64_t first, int64_t n,
                                  const float *q, const float *pred, const double box[3], float *rx, float *ry,
                                  float *rz, hipStream_t s) {
    hipLaunchKernelGGL(k_coarse_residual, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cx, cy, cz, first,
                       n, q, pred, box[0], box[1], box[2], rx, ry, rz);
    return hipGetLastError();
}

// Fine positions: network prediction plus the coarse residuals interpolated
// over the coarse tetrahedron that contains the vertex's Lagrangian point;
// coarse vertices keep their data exactly.
__global__ void k_place_hybrid(const float *__restrict__ cx, const float *__restrict__ cy,
                               const float *__restrict__ cz, const float *__restrict__ rx,
                               const float *__restrict__ ry, const float *__restrict__ rz, int d0, int d1,
                               int d2, int r, int64_t first, int64_t n, const float *__restrict__ q,
                               const float *__restrict__ pred, double L0, double L1, double L2,
                               float *__restrict__ fx, float *__restrict__ fy, float *__restrict__ fz) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int64_t id = first + j;
    const int f0 = d0 * r, f1 = d1 * r;
    const int I = (int)(id % f0), J = (int)((id / f0) % f1), K = (int)(id / ((int64_t)f0 * f1));
    const int i = I / r, jj0 = J / r, k = K / r;
    if (I % r == 0 && J % r == 0 && K % r == 0) {
        const int64_t c = (int64_t)i + (int64_t)d0 * (jj0 + (int64_t)d1 * k);
        fx[id] = cx[c];
        fy[id] = cy[c];
        fz[id] = cz[c];
        return;
    }
    const double p[3] = {(double)(I % r) / r, (double)(J % r) / r, (double)(K % r) / r};
    double lam[4];
    const int t = unit_cube_tet(p, lam);
    double res[3] = {0.0, 0.0, 0.0};
    for (int m = 0; m < 4 && t >= 0; ++m) {
        const int c = cube_corner(t, m);
        int ii = i + (c & 1), jj = jj0 + ((c >> 1) & 1), kk = k + ((c >> 2) & 1);
        if (ii == d0) ii = 0;
        if (jj == d1) jj = 0;
        if (kk == d2) kk = 0;
        const int64_t cid = ii + (int64_t)d0 * (jj + (int64_t)d1 * kk);
        res[0] += lam[m] * (double)rx[cid];
        res[1] += lam[m] * (double)ry[cid];
        res[2] += lam[m] * (double)rz[cid];
    }
    fx[id] = wrap_f32(((double)q[3 * j] + (double)pred[3 * j]) * L0 + res[0], L0);
    fy[id] = wrap_f32(((double)q[3 * j + 1] + (double)pred[3 * j + 1]) * L1 + res[1], L1);
    fz[id] = wrap_f32(((double)q[3 * j + 2] + (double)pred[3 * j + 2]) * L2 + res[2], L2);
}

hipError_t launch_place_hybrid(const float *cx, const float *cy, const float *cz, const float *rx,
                               const float *ry, const float *rz, const int cdims[3], int r, int64_t first,
                               int64_t n, const float *q, const float *pred, const double box[3], float *fx,
                               float *fy, float *fz, hipStream_t s) {
    hipLaunchKernelGGL(k_place_hybrid, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cx, cy, cz, rx, ry, rz,
                       cdims[0], cdims[1], cdims[2], r, first, n, q, pred, box[0], box[1], box[2], fx, fy, fz);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace tess
