// Refinement network: constants, parameter layout and kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace tess {
namespace mlp {

constexpr int kWidth = 128;   // hidden width (and number of Fourier features)
constexpr int kFreq = 64;     // Fourier frequencies: features sin and cos of each
constexpr int kDepth = 4;     // hidden layers
constexpr int kSlice = 64;    // batch rows per weight-gradient partial (LDS: 2 x 128 x 72 bf16)
constexpr int kOutPart = 1 + 3 * kWidth + 3;  // loss, dW5, db5 per output block

// Flat FP32 parameter vector: W1 (128 x 128, row = output), b1, ..., W4, b4,
// W5 (3 x 128), b5.
constexpr int64_t kLayerParams = (int64_t)kWidth * kWidth + kWidth;
constexpr int64_t kOffW5 = kDepth * kLayerParams;
constexpr int64_t kOffB5 = kOffW5 + 3 * kWidth;
constexpr int64_t kParams = kOffB5 + 3;
static_assert(kParams == 66435, "parameter count");
__host__ __device__ constexpr int64_t param_offset_W(int l) { return l * kLayerParams; }
__host__ __device__ constexpr int64_t param_offset_b(int l) { return l * kLayerParams + (int64_t)kWidth * kWidth; }

// Where minibatches come from: the coarse lattice's tracers (dims d, box
// lengths L), drawn by a hash of (seed, step, sample).
struct BatchSource {
    const float *x, *y, *z;
    int32_t d[3];
    double L[3];
    uint64_t seed;
};
hipError_t launch_gather_batch(const BatchSource &S, uint64_t step, int64_t nb, float *q, float *target,
                               hipStream_t s);

// Device arrays of a training step of n samples.  Feature-major arrays hold
// ld = train_rows(n) samples per feature, zeros from n on.
__host__ __device__ constexpr int64_t train_rows(int64_t n) { return (n + kSlice - 1) / kSlice * kSlice; }
struct TrainNet {
    float *master, *m, *v;   // parameters and moments
    const float *B;          // Fourier frequencies
    float *q, *target, *pred;  // [n][3]
    __bf16 *Wb, *WTb;        // hidden weights in bf16, row-major and transposed
    __bf16 *act;             // [kDepth + 1][kWidth][ld]: features, H1 .. H4
    __bf16 *err;             // [kDepth][kWidth][ld]: dZ1 .. dZ4
    float *dout;             // [4][ld]: the output's gradient, then the squared error
};
struct AdamStep {
    float lr, b1, a1, b2, a2, eps, c1, c2;
};
AdamStep adam_step(double lr, double b1, double b2, double eps, int t);
// Forward and backward of T.q against T.target: pred, act, err, dout.
hipError_t launch_train_pass(const TrainNet &T, int64_t n, hipStream_t s);
// After it: the gradients into grad[kParams] and the summed squared error
// into *loss (null: not wanted); or the Adam update of T's parameters, and
// the minibatch of step `next` (0: none) into T.q and T.target.
hipError_t launch_train_grads(const TrainNet &T, int64_t n, float *grad, float *loss, hipStream_t s);
hipError_t launch_train_update(const TrainNet &T, int64_t n, const AdamStep &A, float *loss, const BatchSource &S,
                               uint64_t next, hipStream_t s);
hipError_t launch_adam(float *w, float *m, float *v, const float *g, int64_t count, const AdamStep &A, hipStream_t s);
hipError_t launch_cast_weights(const float *master, __bf16 *Wb, __bf16 *WTb, hipStream_t s);
// Inference: pred[n][3] from q[n][3] in one pass (features, hidden layers
// and output layer per 16-sample tile in registers; bf16 operands rounded
// from the FP32 master parameters, FP32 accumulation).  `master` is read 16
// bytes at a time: the start of an allocation.
hipError_t launch_mlp_infer(const float *q, int64_t n, const float *B, const float *master, float *pred,
                            hipStream_t s);

}  // namespace mlp
}  // namespace tess

namespace tess {
namespace mlp {
hipError_t launch_fine_q(int64_t first, int64_t n, const int fdims[3], float *q, hipStream_t s);
hipError_t launch_place_mlp(const float *cx, const float *cy, const float *cz, const int cdims[3], int r,
                            int64_t first, int64_t n, const float *q, const float *pred,
                            const double box[3], const int fdims[3], float *fx, float *fy, float *fz,
                            hipStream_t s);
// Residuals x - (q + s(q)) L of the network at coarse tracers first..first+n-1.
hipError_t launch_coarse_residual(const float *cx, const float *cy, const float *cz, int64_t first, int64_t n,
                                  const float *q, const float *pred, const double box[3], float *rx, float *ry,
                                  float *rz, hipStream_t s);
// Fine positions first..first+n-1: (q + s(q)) L plus the coarse residuals
// interpolated over the containing coarse tetrahedron.
hipError_t launch_place_hybrid(const float *cx, const float *cy, const float *cz, const float *rx,
                               const float *ry, const float *rz, const int cdims[3], int r, int64_t first,
                               int64_t n, const float *q, const float *pred, const double box[3], float *fx,
                               float *fy, float *fz, hipStream_t s);
hipError_t launch_place_linear(const float *cx, const float *cy, const float *cz, const int cdims[3], int r,
                               const double box[3], float *fx, float *fy, float *fz, hipStream_t s);
}  // namespace mlp
}  // namespace tess
