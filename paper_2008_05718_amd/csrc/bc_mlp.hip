// bc_mlp.hip -- the level-policy network: 5 features -> 32 -> 32 -> 9,
// ReLU hidden layers, FP32.  Training kernels (forward, backward, Adam) and
// batch prediction.  The same weights drive the per-level choice inside the
// step kernels (choose_variant in bc_common.h).
//
// Loss over n samples (x_i, y_i, mask_i), y_ij = log2 of the measured time of
// choice j at that level (three discover variants, three summation options of the
// path-count step and three of the backward step), mask_ij = 1 when it was measured:
//     L = sum_ij mask_ij (f(x_i)_j - y_ij)^2 / (2 * sum_ij mask_ij).
// Gradients are sums over tiles of samples in a fixed order, so they do not
// depend on anything but the samples.
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/bc.h"
#include "bc_dev.h"

namespace bcx {

constexpr int kIn = kMlpIn, kH = kMlpH, kOut = kMlpOut;
constexpr int oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kOut * kH, kP = oB3 + kOut;
static_assert(kP == kMlpParams, "parameter layout");

// Loss and gradient in two launches.  mlp_tiles takes tiles of kTile samples
// per workgroup: forward and backward of the tile (a wavefront computes 8 of the
// 32 hidden units for 64 samples at a time; the weights of a unit are
// wavefront-uniform), then the tile's share of the gradient, a contraction over
// its samples: D1^T [X 1], D2^T H1 and D3^T H2 on the FP32 matrix cores, one
// product per wavefront, the remaining bias sums on the fourth.  The
// accumulators stay in registers from tile to tile; every workgroup writes one
// partial gradient, and mlp_combine adds the partials in workgroup order and
// scales them (mlp_scale).  The partition depends only on
// the number of samples, so the same samples give the same bits.
//
// What bounds it: the latency of the two launches and of one tile's dependent
// layers.  4096 samples: 22 us a call, against 1.38 ms for one thread per
// parameter walking all samples in order; the error against 64 bits falls
// from 6e-7 to 1e-7, the sums being shorter.
constexpr int kTile = 64;
constexpr int kStride = kTile + 1;  // LDS rows of a unit's values: no bank conflicts across units
constexpr int kMaxTiles = 256;      // workgroups of mlp_tiles
constexpr int kPart = kP + 2;       // partial gradient, loss, measured targets (a whole number in the last word)
typedef float f32x16 __attribute__((ext_vector_type(16)));

// The loss is a mean, and a sum over all samples may leave FP32 where the mean
// does not.  So every error is taken times 2^-k, the power of two at or below
// 1 / (targets of all samples), from the start, and the sums times 2^k / (targets measured).
// (A power of two changes no rounding.)
static int mlp_scale(int64_t n) {
    int k = 0;
    while (k < 62 && ((int64_t)1 << k) < n * kOut) ++k;
    return k;
}

static int mlp_blocks(int64_t n) { return (int)std::min<int64_t>((n + kTile - 1) / kTile, kMaxTiles); }

__global__ __launch_bounds__(256) void mlp_tiles(const float *__restrict__ w, const float *__restrict__ X,
                                                 const float *__restrict__ Y, const uint8_t *__restrict__ mask,
                                                 int64_t n, float scale, float *__restrict__ part) {
    __shared__ float sx[(kIn + 1) * kStride];  // features, and a row of ones
    __shared__ float h1[kH * kStride], h2[kH * kStride], d1[kH * kStride], d2[kH * kStride], d3[kOut * kStride];
    __shared__ float se[4 * kTile];
    __shared__ unsigned sc[4 * kTile];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int row = lane & 31, half = lane >> 5;
    f32x16 acc = {};
    float bias = 0.0f, loss = 0.0f;
    unsigned count = 0;  // (a workgroup has n / 256 samples: below 2^32 up to 10^11)
    for (int64_t base = (int64_t)blockIdx.x * kTile; base < n; base += (int64_t)gridDim.x * kTile) {
        // samples beyond the last one repeat it with nothing measured
        const int64_t r = min(base + lane, n - 1);
        const bool on = base + lane < n;
        float x[kIn];
#pragma unroll
        for (int i = 0; i < kIn; ++i) x[i] = X[r * kIn + i];
        if (wv == 0) {
#pragma unroll
            for (int i = 0; i < kIn; ++i) sx[i * kStride + lane] = x[i];
            sx[kIn * kStride + lane] = 1.0f;
        }
        for (int j = 8 * wv; j < 8 * wv + 8; ++j) {
            float s = w[oB1 + j];
#pragma unroll
            for (int i = 0; i < kIn; ++i) s += w[oW1 + j * kIn + i] * x[i];
            h1[j * kStride + lane] = fmaxf(s, 0.0f);
        }
        __syncthreads();
        {
            float s[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] = w[oB2 + 8 * wv + j];
            for (int i = 0; i < kH; ++i) {
                const float h = h1[i * kStride + lane];
#pragma unroll
                for (int j = 0; j < 8; ++j) s[j] += w[oW2 + (8 * wv + j) * kH + i] * h;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) h2[(8 * wv + j) * kStride + lane] = fmaxf(s[j], 0.0f);
        }
        __syncthreads();
        float e = 0.0f;
        unsigned c = 0;
        for (int k = wv; k < kOut; k += 4) {
            float s = w[oB3 + k];
            for (int i = 0; i < kH; ++i) s += w[oW3 + k * kH + i] * h2[i * kStride + lane];
            const bool m = on && mask[r * kOut + k] != 0;
            const float diff = m ? s - Y[r * kOut + k] : 0.0f;
            const float d = diff * scale;
            d3[k * kStride + lane] = d;
            e += d * diff;
            c += m ? 1u : 0u;
        }
        se[wv * kTile + lane] = 0.5f * e;
        sc[wv * kTile + lane] = c;
        __syncthreads();
        {
            float s[8] = {};
            for (int k = 0; k < kOut; ++k) {
                const float d = d3[k * kStride + lane];
#pragma unroll
                for (int j = 0; j < 8; ++j) s[j] += w[oW3 + k * kH + 8 * wv + j] * d;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int at = (8 * wv + j) * kStride + lane;
                d2[at] = h2[at] > 0.0f ? s[j] : 0.0f;
            }
        }
        __syncthreads();
        {
            float s[8] = {};
            for (int k = 0; k < kH; ++k) {
                const float d = d2[k * kStride + lane];
#pragma unroll
                for (int j = 0; j < 8; ++j) s[j] += w[oW2 + k * kH + 8 * wv + j] * d;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int at = (8 * wv + j) * kStride + lane;
                d1[at] = h1[at] > 0.0f ? s[j] : 0.0f;
            }
        }
        __syncthreads();
        if (wv < 3) {
            // A[row][sample] x B[sample][column], two samples per instruction
            const float *A = wv == 0 ? d1 : (wv == 1 ? d2 : d3), *B = wv == 0 ? sx : (wv == 1 ? h1 : h2);
            const bool ar = wv < 2 || row < kOut, bc = wv > 0 || row <= kIn;
#pragma unroll 8
            for (int k = 0; k < kTile; k += 2) {
                const int at = row * kStride + k + half;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ar ? A[at] : 0.0f, bc ? B[at] : 0.0f, acc, 0, 0, 0);
            }
        } else if (lane < kH + kOut) {
            const float *D = lane < kH ? d2 + lane * kStride : d3 + (lane - kH) * kStride;
            float t = 0.0f;
            for (int k = 0; k < kTile; ++k) t += D[k];
            bias += t;
        } else if (lane < kH + kOut + 8) {  // loss and targets, 64 of the 256 values per lane
            const int q = lane - (kH + kOut), at = (q & 3) * kTile;
            float t = 0.0f;
            unsigned u = 0;
            for (int k = 0; k < kTile; ++k) {
                t += se[at + k];
                u += sc[at + k];
            }
            if (q < 4) loss += t;
            else count += u;
        }
        __syncthreads();
    }
    float *p = part + (size_t)blockIdx.x * kPart;
    if (wv < 3) {
        // accumulator i of a lane: column lane & 31, row 8 (i / 4) + 4 (lane / 32) + i % 4
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int j = 8 * (i >> 2) + 4 * half + (i & 3);
            if (wv == 0) {
                if (row < kIn) p[oW1 + j * kIn + row] = acc[i];
                else if (row == kIn) p[oB1 + j] = acc[i];
            } else if (wv == 1) {
                p[oW2 + j * kH + row] = acc[i];
            } else if (j < kOut) {
                p[oW3 + j * kH + row] = acc[i];
            }
        }
    } else {
        const float l4 = __shfl(loss, kH + kOut) + __shfl(loss, kH + kOut + 1) + __shfl(loss, kH + kOut + 2) +
                         __shfl(loss, kH + kOut + 3);
        const unsigned c4 = __shfl(count, kH + kOut + 4) + __shfl(count, kH + kOut + 5) + __shfl(count, kH + kOut + 6) +
                            __shfl(count, kH + kOut + 7);
        if (lane < kH) p[oB2 + lane] = bias;
        else if (lane < kH + kOut) p[oB3 + lane - kH] = bias;
        else if (lane == kH + kOut) p[kP] = l4;
        else if (lane == kH + kOut + 1) p[kP + 1] = __uint_as_float(c4);
    }
}

// Adam (Kingma & Ba), step t >= 1.
struct AdamArgs {
    float *w = nullptr, *m1 = nullptr, *m2 = nullptr;  // w == nullptr: no update
    int t = 0;
    float lr = 0.0f, b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
};

// Sum of the partials, workgroup by workgroup, one thread per parameter (8
// loads in flight); thread kP sums the loss.  With adam.w the weights are
// updated by the same thread.  The measured targets are counted in whole
// numbers; none measured: loss and gradient are zero.
__global__ __launch_bounds__(64) void mlp_combine(const float *__restrict__ part, int blocks, double unscale,
                                                  float *__restrict__ grad, float *__restrict__ loss, AdamArgs adam) {
    __shared__ unsigned long long s_cnt[64];
    unsigned long long c = 0;
    for (int b = threadIdx.x; b < blocks; b += 64) c += __float_as_uint(part[(size_t)b * kPart + kP + 1]);
    s_cnt[threadIdx.x] = c;
    __syncthreads();
    unsigned long long total = 0;
    for (int i = 0; i < 64; ++i) total += s_cnt[i];
    const float inv = total ? (float)(unscale / (double)total) : 0.0f;
    const int p = blockIdx.x * 64 + threadIdx.x;
    if (p > kP) return;
    float g = 0.0f;
    int b = 0;
    for (; b + 8 <= blocks; b += 8) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = part[(size_t)(b + q) * kPart + p];
#pragma unroll
        for (int q = 0; q < 8; ++q) g += v[q];
    }
    for (; b < blocks; ++b) g += part[(size_t)b * kPart + p];
    g *= inv;
    if (p == kP) {
        *loss = g;
        return;
    }
    grad[p] = g;
    if (!adam.w) return;
    const float a = adam.b1 * adam.m1[p] + (1.0f - adam.b1) * g;
    const float v = adam.b2 * adam.m2[p] + (1.0f - adam.b2) * g * g;
    adam.m1[p] = a;
    adam.m2[p] = v;
    const float ah = a / (1.0f - powf(adam.b1, (float)adam.t));
    const float vh = v / (1.0f - powf(adam.b2, (float)adam.t));
    adam.w[p] -= adam.lr * ah / (sqrtf(vh) + adam.eps);
}

__global__ void mlp_predict(const float *__restrict__ w, const float *__restrict__ X, int64_t n,
                            float *__restrict__ Y) {
    __shared__ float sw[kP];
    for (int i = threadIdx.x; i < kP; i += blockDim.x) sw[i] = w[i];
    __syncthreads();
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        float x[kIn], h1[kH], h2[kH];
        for (int i = 0; i < kIn; ++i) x[i] = X[r * kIn + i];
        for (int j = 0; j < kH; ++j) {
            float s = sw[oB1 + j];
            for (int i = 0; i < kIn; ++i) s += sw[oW1 + j * kIn + i] * x[i];
            h1[j] = fmaxf(s, 0.0f);
        }
        for (int j = 0; j < kH; ++j) {
            float s = sw[oB2 + j];
            for (int i = 0; i < kH; ++i) s += sw[oW2 + j * kH + i] * h1[i];
            h2[j] = fmaxf(s, 0.0f);
        }
        for (int k = 0; k < kOut; ++k) {
            float s = sw[oB3 + k];
            for (int i = 0; i < kH; ++i) s += sw[oW3 + k * kH + i] * h2[i];
            Y[r * kOut + k] = s;
        }
    }
}

}  // namespace bcx

using namespace bcx;

namespace {

// Device buffers for one training / gradient call.
struct MlpBufs {
    float *w = nullptr, *X = nullptr, *Y = nullptr, *part = nullptr, *grad = nullptr, *m1 = nullptr, *m2 = nullptr,
          *loss = nullptr;
    uint8_t *mask = nullptr;
    bool owned = true;  // false: views into the static scratch (nothing to free)
    ~MlpBufs() {
        if (!owned) return;
        void *ps[] = {w, X, Y, part, grad, m1, m2, loss, mask};
        for (void *p : ps)
            if (p) (void)hipFree(p);
    }
};

}  // namespace

// Records the thread-local error text (bc_api.hip) and returns s.
bc_status bc_set_error(bc_status s, const char *msg);

#define MLP_TRY(expr)                                                                 \
    do {                                                                              \
        hipError_t _e = (expr);                                                       \
        if (_e != hipSuccess)                                                         \
            return bc_set_error(_e == hipErrorOutOfMemory ? BC_ERR_OUT_OF_MEMORY : BC_ERR_DEVICE, \
                                (std::string(#expr) + ": " + hipGetErrorString(_e)).c_str()); \
    } while (0)

static bc_status mlp_upload(MlpBufs &b, const float *weights, const float *X, const float *Y, const uint8_t *mask,
                            int64_t n, hipStream_t st) {
    const size_t N = (size_t)(n > 0 ? n : 1);
    MLP_TRY(hipMalloc((void **)&b.w, kP * sizeof(float)));
    MLP_TRY(hipMalloc((void **)&b.X, N * kIn * sizeof(float)));
    MLP_TRY(hipMalloc((void **)&b.Y, N * kOut * sizeof(float)));
    MLP_TRY(hipMalloc((void **)&b.mask, N * kOut));
    MLP_TRY(hipMalloc((void **)&b.part, (size_t)mlp_blocks((int64_t)N) * kPart * sizeof(float)));
    MLP_TRY(hipMalloc((void **)&b.grad, kP * sizeof(float)));
    MLP_TRY(hipMalloc((void **)&b.m1, kP * sizeof(float)));
    MLP_TRY(hipMalloc((void **)&b.m2, kP * sizeof(float)));
    MLP_TRY(hipMalloc((void **)&b.loss, sizeof(float)));
    MLP_TRY(hipMemcpyAsync(b.w, weights, kP * sizeof(float), hipMemcpyHostToDevice, st));
    if (n > 0) {
        MLP_TRY(hipMemcpyAsync(b.X, X, (size_t)n * kIn * sizeof(float), hipMemcpyHostToDevice, st));
        MLP_TRY(hipMemcpyAsync(b.Y, Y, (size_t)n * kOut * sizeof(float), hipMemcpyHostToDevice, st));
        MLP_TRY(hipMemcpyAsync(b.mask, mask, (size_t)n * kOut, hipMemcpyHostToDevice, st));
    }
    return BC_OK;
}

static bc_status mlp_check(const float *weights, const float *X, const float *Y, const uint8_t *mask, int64_t n) {
    if (!weights || n < 1 || !X || !Y || !mask) return bc_set_error(BC_ERR_INVALID_ARG, "NULL argument or n < 1");
    int64_t cnt = 0;
    for (int64_t i = 0; i < n * kOut; ++i) cnt += mask[i] ? 1 : 0;
    if (cnt == 0) return bc_set_error(BC_ERR_INVALID_ARG, "no measured targets (mask is all zero)");
    for (int64_t i = 0; i < n * kIn; ++i)
        if (!std::isfinite(X[i])) return bc_set_error(BC_ERR_INVALID_ARG, "non-finite feature");
    for (int64_t i = 0; i < n * kOut; ++i)
        if (mask[i] && !std::isfinite(Y[i])) return bc_set_error(BC_ERR_INVALID_ARG, "non-finite target");
    return BC_OK;
}

static void mlp_step_grad(MlpBufs &b, int64_t n, hipStream_t st, const AdamArgs &adam = AdamArgs{}) {
    const int blocks = mlp_blocks(n);
    const int k = mlp_scale(n);
    mlp_tiles<<<blocks, 256, 0, st>>>(b.w, b.X, b.Y, b.mask, n, std::ldexp(1.0f, -k), b.part);
    mlp_combine<<<(kP + 1 + 63) / 64, 64, 0, st>>>(b.part, blocks, std::ldexp(1.0, k), b.grad, b.loss, adam);
}

extern "C" bc_status bc_mlp_loss_grad(const float *weights, const float *X, const float *Y, const uint8_t *mask,
                                      int64_t n, float *loss, float *grad, void *stream) {
    bc_status s = mlp_check(weights, X, Y, mask, n);
    if (s != BC_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    MlpBufs b;
    s = mlp_upload(b, weights, X, Y, mask, n, st);
    if (s != BC_OK) return s;
    mlp_step_grad(b, n, st);
    MLP_TRY(hipGetLastError());
    float l = 0.0f;
    std::vector<float> g(kP);
    MLP_TRY(hipMemcpyAsync(&l, b.loss, sizeof(float), hipMemcpyDeviceToHost, st));
    MLP_TRY(hipMemcpyAsync(g.data(), b.grad, kP * sizeof(float), hipMemcpyDeviceToHost, st));
    MLP_TRY(hipStreamSynchronize(st));
    if (loss) *loss = l;
    if (grad) std::memcpy(grad, g.data(), kP * sizeof(float));
    return BC_OK;
}

// ------------------------------------------------ allocation-free variant
// bc_mlp_loss_grad_noalloc keeps the partial gradients, losses and target
// counts in this fixed array: no device memory is allocated per call.  Each GPU holds its own copy for the life of the process.  Host code
// must not pass the array's name to a kernel (on the host it only stands for
// the symbol): the device address comes from hipGetSymbolAddress, taken once
// per device on the first call there.
constexpr int64_t kNoAllocMaxSamples = 16384;
constexpr size_t kNoAllocFloats = (size_t)kMaxTiles * kPart;
static __device__ __align__(256) float scratch[kNoAllocFloats];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

static bc_status scratch_address(float **out) {
    int dev = -1;
    MLP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return bc_set_error(BC_ERR_NOT_SUPPORTED, "device index beyond 63");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        MLP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return bc_set_error(BC_ERR_DEVICE, "hipGetSymbolAddress returned NULL for the scratch array");
        g_scratch_ptr[dev] = (float *)p;
    }
    *out = g_scratch_ptr[dev];
    return BC_OK;
}

extern "C" bc_status bc_mlp_loss_grad_noalloc(const float *weights, const float *X, const float *Y,
                                              const uint8_t *mask, int64_t n, float *loss, float *grad,
                                              void *stream) {
    if (!weights || !X || !Y || !mask || !loss || !grad) return bc_set_error(BC_ERR_INVALID_ARG, "NULL argument");
    if (n < 1 || n > kNoAllocMaxSamples)
        return bc_set_error(BC_ERR_INVALID_ARG, ("n must be in [1, " + std::to_string(kNoAllocMaxSamples) +
                                                 "] for the allocation-free call").c_str());
    float *sc = nullptr;
    bc_status s = scratch_address(&sc);
    if (s != BC_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    MlpBufs b;
    b.owned = false;
    b.w = const_cast<float *>(weights);
    b.X = const_cast<float *>(X);
    b.Y = const_cast<float *>(Y);
    b.mask = const_cast<uint8_t *>(mask);
    b.grad = grad;
    b.loss = loss;
    b.part = sc;
    mlp_step_grad(b, n, st);
    MLP_TRY(hipGetLastError());
    return BC_OK;
}

extern "C" bc_status bc_mlp_train(float *weights, const float *X, const float *Y, const uint8_t *mask, int64_t n,
                                  int32_t steps, float lr, float *final_loss, void *stream) {
    bc_status s = mlp_check(weights, X, Y, mask, n);
    if (s != BC_OK) return s;
    if (steps < 0 || !(lr > 0.0f) || !std::isfinite(lr)) return bc_set_error(BC_ERR_INVALID_ARG, "bad steps or lr");
    for (int i = 0; i < kP; ++i)
        if (!std::isfinite(weights[i])) return bc_set_error(BC_ERR_INVALID_ARG, "non-finite initial weight");
    hipStream_t st = (hipStream_t)stream;
    MlpBufs b;
    s = mlp_upload(b, weights, X, Y, mask, n, st);
    if (s != BC_OK) return s;
    MLP_TRY(hipMemsetAsync(b.m1, 0, kP * sizeof(float), st));
    MLP_TRY(hipMemsetAsync(b.m2, 0, kP * sizeof(float), st));
    AdamArgs adam;
    adam.w = b.w;
    adam.m1 = b.m1;
    adam.m2 = b.m2;
    adam.lr = lr;
    for (adam.t = 1; adam.t <= steps; ++adam.t) mlp_step_grad(b, n, st, adam);
    mlp_step_grad(b, n, st);  // loss of the final weights
    MLP_TRY(hipGetLastError());
    std::vector<float> w(kP);
    float l = 0.0f;
    MLP_TRY(hipMemcpyAsync(w.data(), b.w, kP * sizeof(float), hipMemcpyDeviceToHost, st));
    MLP_TRY(hipMemcpyAsync(&l, b.loss, sizeof(float), hipMemcpyDeviceToHost, st));
    MLP_TRY(hipStreamSynchronize(st));
    for (int i = 0; i < kP; ++i)
        if (!std::isfinite(w[i])) return bc_set_error(BC_ERR_DEVICE, "training diverged (non-finite weights)");
    std::memcpy(weights, w.data(), kP * sizeof(float));
    if (final_loss) *final_loss = l;
    return BC_OK;
}

extern "C" bc_status bc_mlp_predict(const float *weights, const float *X, int64_t n, float *Y, void *stream) {
    if (!weights || !X || !Y || n < 0) return bc_set_error(BC_ERR_INVALID_ARG, "NULL argument or n < 0");
    if (n == 0) return BC_OK;
    hipStream_t st = (hipStream_t)stream;
    float *dw = nullptr, *dx = nullptr, *dy = nullptr;
    auto cleanup = [&]() {
        if (dw) (void)hipFree(dw);
        if (dx) (void)hipFree(dx);
        if (dy) (void)hipFree(dy);
    };
    hipError_t e = hipMalloc((void **)&dw, kP * sizeof(float));
    if (e == hipSuccess) e = hipMalloc((void **)&dx, (size_t)n * kIn * sizeof(float));
    if (e == hipSuccess) e = hipMalloc((void **)&dy, (size_t)n * kOut * sizeof(float));
    if (e == hipSuccess) e = hipMemcpyAsync(dw, weights, kP * sizeof(float), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(dx, X, (size_t)n * kIn * sizeof(float), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) {
        mlp_predict<<<(int)std::min<int64_t>((n + 255) / 256, 4096), 256, 0, st>>>(dw, dx, n, dy);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(Y, dy, (size_t)n * kOut * sizeof(float), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    cleanup();
    if (e != hipSuccess) return bc_set_error(BC_ERR_DEVICE, hipGetErrorString(e));
    return BC_OK;
}
