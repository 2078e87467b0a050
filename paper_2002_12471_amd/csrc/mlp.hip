// Scatter-surrogate network on gfx950: 8 -> 128 -> 128 -> 128 -> 1 with GELU
// (tanh form), bf16 weights and activations, FP32 accumulation (MFMA), FP32
// master weights and Adam.
//
// Every matrix product is C[m][n] = sum_k A[m][k] Bt[n][k], with both operands
// row-major bf16 and contiguous in k, which is the operand layout of
// v_mfma_f32_16x16x16_bf16 (lane l holds A[l%16][4(l/16)..+3] and
// B[4(l/16)..+3][l%16]; D[4(l/16)+v][l%16] comes back in register v):
//   forward       Z[b][out]  = H[b][in]   . Wt[out][in]
//   data grad     dH[b][in]  = D[b][out]  . W[in][out]
//   weight grad   dW[in][out] = Ht[in][b] . Dt[out][b]
// A training step is three kernels: forward and data gradients of 16 samples
// per workgroup (k_train), the weight and bias gradients in slices of the
// batch (k_weight_grads), and the sum of the slices (k_sum_grads).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <vector>

#include "lmosem_int.h"
#include "mlp_infer.h"

namespace lmo {

typedef short bf16x4 __attribute__((ext_vector_type(4)));

__device__ __host__ inline uint16_t f2bf(float f) {
    uint32_t u;
    memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest, ties to even
    return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

constexpr float kGeluC = 0.7978845608028654f;   // sqrt(2/pi)
constexpr float kGeluA = 0.044715f;

__device__ inline float gelu(float x) {
    const float u = kGeluC * (x + kGeluA * x * x * x);
    return 0.5f * x * (1.0f + tanhf(u));
}
__device__ inline float gelu_grad(float x) {
    const float u = kGeluC * (x + kGeluA * x * x * x);
    const float t = tanhf(u);
    return 0.5f * (1.0f + t) + 0.5f * x * (1.0f - t * t) * kGeluC * (1.0f + 3.0f * kGeluA * x * x);
}

// ---------------------------------------------------------------- network state
// Parameter order (flat FP32 master copy): W1[8][128] b1[128] W2[128][128] b2
// W3[128][128] b3 W4[128][1] b4[1]; W[in][out].
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kIn * kHid, kOffW2 = kOffB1 + kHid, kOffB2 = kOffW2 + kHid * kHid,
              kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kHid * kHid, kOffW4 = kOffB3 + kHid,
              kOffB4 = kOffW4 + kHid, kNParams = kOffB4 + 1;
static_assert(kNParams == 34305, "parameter count");

struct NetBf16 {
    uint16_t *w1t, *w2t, *w3t;   // [out][in] (w1t: [128][16] zero-padded)
    uint16_t *w2, *w3;           // [in][out]
    uint16_t *w4;                // [128]
};

// master FP32 -> bf16 copies in both layouts
__global__ void k_pack(const float *__restrict__ p, NetBf16 nb) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < kHid * kInPad) {   // w1t[out][in]
        const int o = idx / kInPad, i = idx % kInPad;
        nb.w1t[idx] = i < kIn ? f2bf(p[kOffW1 + i * kHid + o]) : 0;
    }
    if (idx < kHid * kHid) {
        const int a = idx / kHid, b = idx % kHid;   // idx = a*128 + b
        nb.w2[idx] = f2bf(p[kOffW2 + idx]);          // [in a][out b]
        nb.w3[idx] = f2bf(p[kOffW3 + idx]);
        nb.w2t[idx] = f2bf(p[kOffW2 + b * kHid + a]);   // [out a][in b]
        nb.w3t[idx] = f2bf(p[kOffW3 + b * kHid + a]);
    }
    if (idx < kHid) nb.w4[idx] = f2bf(p[kOffW4 + idx]);
}

// what the weight gradients read, transposed bf16 [unit][n], and the batch's
// output gradients
struct Transposed {
    uint16_t *xt;                 // [16][n], inputs zero-padded
    uint16_t *h1t, *h2t, *h3t;    // [128][n]
    uint16_t *d1t, *d2t, *d3t;    // [128][n]
    float *dy;                    // [n]
};

enum class Step { outputs, gradient, train };   // y alone; from given dy; from targets

// One step of 16 samples, one workgroup: wave w holds hidden units 16 w .. 16 w
// + 15 of every layer, a lane one unit and four samples (4 q + v).  Activations
// and deltas pass through LDS to be the next product's A operand, the weights
// come from the L2 as they are (32 KB a matrix; the next matrix is on its way
// while the current layer's GELU is evaluated), pre-activations never leave the
// registers (their GELU slopes do the rest), and what the weight gradients need
// is written transposed, 8 bytes a lane.  A chain of six layers on one workgroup
// per compute unit bounds it: 18 us for 4096 samples (20 with four waves of 32
// units), where 12 kernels that passed 30 MB through memory took 83 us.
constexpr int kRows = 16;
constexpr int kTrainThreads = 64 * kHid / 16;

template <Step STEP>
__global__ __launch_bounds__(kTrainThreads) void k_train(const float *__restrict__ X, const float *__restrict__ p,
                                                         NetBf16 nb, int n, const float *__restrict__ dy_in,
                                                         const float *__restrict__ target, float inv_total,
                                                         float *__restrict__ y, Transposed tr,
                                                         double *__restrict__ loss_part) {
    typedef uint16_t Rows[kHid + 8];
    __shared__ __align__(16) Rows act[2][kRows];
    __shared__ float dy_s[kRows];
    __shared__ double loss_s[kRows];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4, b0 = blockIdx.x * kRows;
    const int unit = 16 * wave + r;
    constexpr int kSteps = kHid / 16;
    bf16x4 w[kSteps];
    auto weights = [&](const uint16_t *Bt) {
#pragma unroll
        for (int k = 0; k < kSteps; ++k) w[k] = *reinterpret_cast<const bf16x4 *>(Bt + unit * kHid + 16 * k + 4 * q);
    };
    f32x4 acc;
    auto product = [&](const Rows *A) {
        acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kSteps; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4 *>(&A[r][16 * k + 4 * q]), w[k], acc,
                                                            0, 0, 0);
    };
    // the lane's unit, samples 4 q + v: to LDS, and transposed to memory
    auto put = [&](Rows *A, uint16_t *out, const uint16_t (&v)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) A[4 * q + i][unit] = v[i];
        if (STEP != Step::outputs) {
            const bf16x4 x = {(short)v[0], (short)v[1], (short)v[2], (short)v[3]};
            *reinterpret_cast<bf16x4 *>(out + (size_t)unit * n + b0 + 4 * q) = x;
        }
        __syncthreads();
    };
    // inputs, zero-padded to 16
    if (threadIdx.x < kRows * kInPad) {
        const int b = threadIdx.x >> 4, i = threadIdx.x & 15;
        act[0][b][i] = i < kIn ? f2bf(X[(size_t)(b0 + b) * kIn + i]) : 0;
        // (transposed: a row per 16 threads)
        if (STEP != Step::outputs) tr.xt[(size_t)b * n + b0 + i] = b < kIn ? f2bf(X[(size_t)(b0 + i) * kIn + b]) : 0;
    }
    const bf16x4 w1 = *reinterpret_cast<const bf16x4 *>(nb.w1t + unit * kInPad + 4 * q);
    weights(nb.w2t);
    __syncthreads();
    float slope[3][4];
    auto layer = [&](int l, const float *bias, Rows *A, uint16_t *out) {
        const float bj = bias[unit];
        uint16_t h[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float z = acc[v] + bj;
            h[v] = f2bf(gelu(z));
            slope[l][v] = gelu_grad(z);
        }
        put(A, out, h);
    };
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4 *>(&act[0][r][4 * q]), w1,
                                                    f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    layer(0, p + kOffB1, act[1], tr.h1t);
    product(act[1]);
    weights(nb.w3t);
    layer(1, p + kOffB2, act[0], tr.h2t);
    product(act[0]);
    weights(nb.w3);
    layer(2, p + kOffB3, act[1], tr.h3t);
    if (STEP == Step::gradient) {
        if (threadIdx.x < kRows) dy_s[threadIdx.x] = dy_in[b0 + threadIdx.x];
    } else if (threadIdx.x < kRows) {
        const int b = threadIdx.x;
        float s = 0.0f;
        for (int k = 0; k < kHid; ++k) s = fmaf(bf2f(act[1][b][k]), bf2f(nb.w4[k]), s);
        s += p[kOffB4];
        if (STEP == Step::outputs) {
            y[b0 + b] = s;
        } else {   // mean squared error
            const float e = s - target[b0 + b];
            dy_s[b] = 2.0f * e * inv_total;
            loss_s[b] = (double)e * e;
        }
    }
    if (STEP == Step::outputs) return;
    __syncthreads();
    if (threadIdx.x < kRows) tr.dy[b0 + threadIdx.x] = dy_s[threadIdx.x];
    if (STEP == Step::train && threadIdx.x == 0) {
        double l = 0.0;
        for (int b = 0; b < kRows; ++b) l += loss_s[b];
        loss_part[blockIdx.x] = l;
    }
    // deltas d[b][k] = dh[b][k] gelu'(z[b][k]), the last layer's dh from the output row
    uint16_t d[4];
    const float w4 = bf2f(nb.w4[unit]);
#pragma unroll
    for (int v = 0; v < 4; ++v) d[v] = f2bf(dy_s[4 * q + v] * w4 * slope[2][v]);
    put(act[0], tr.d3t, d);
    auto delta = [&](int l, Rows *A, uint16_t *out) {
#pragma unroll
        for (int v = 0; v < 4; ++v) d[v] = f2bf(acc[v] * slope[l][v]);
        put(A, out, d);
    };
    product(act[0]);
    weights(nb.w2);
    delta(1, act[1], tr.d2t);
    product(act[1]);
    delta(0, act[0], tr.d1t);
}

// Weight gradients dW[in][out] = sum_b Ht[in][b] Dt[out][b] and the bias
// gradients, in one launch: the products have few output blocks and a long K
// (the batch), so they are split over K into slices whose partial products
// k_sum_grads adds in a fixed order; the bias sums fill the rest of the chip
// meanwhile.  A 64x64 block per workgroup, 32x32 per wave (2x2 MFMA tiles).
constexpr int kSplitMax = 32;   // slices of one product
constexpr int kPartial = 2 * kHid * kHid + kInPad * kHid;   // one slice of all three products: W3, W2, W1 (padded)

// slices of a batch of n: at least 256 samples each
static int grad_slices(int n, int &slice) {
    const int s = std::max(1, std::min(kSplitMax, n / 256));
    slice = ((n + s - 1) / s + 15) / 16 * 16;
    return (n + slice - 1) / slice;
}

__global__ __launch_bounds__(256) void k_weight_grads(Transposed tr, int n, int slices, int slice,
                                                      float *__restrict__ part, float *__restrict__ g) {
    __shared__ float red[256];
    const int blocks = 10 * slices;   // W3: 4 blocks of 64 x 64, W2: 4, W1 (16 rows): 2
    if ((int)blockIdx.x < blocks) {
        const int z = blockIdx.x / 10, job = blockIdx.x - 10 * z;
        const uint16_t *A = job < 4 ? tr.h2t : job < 8 ? tr.h1t : tr.xt;
        const uint16_t *Bt = job < 4 ? tr.d3t : job < 8 ? tr.d2t : tr.d1t;
        float *C = part + (size_t)z * kPartial + (job < 4 ? 0 : job < 8 ? kHid * kHid : 2 * kHid * kHid);
        const int M = job < 8 ? kHid : kInPad;
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, kq = (lane >> 4) * 4;
        const int m_base = (job < 8 ? (job & 3) >> 1 : 0) * 64 + (wave >> 1) * 32, n_base = (job & 1) * 64 + (wave & 1) * 32;
        if (m_base >= M) return;
        f32x4 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        const uint16_t *a0 = A + (size_t)(m_base + r) * n + kq, *a1 = m_base + 16 < M ? a0 + (size_t)16 * n : a0;
        const uint16_t *c0 = Bt + (size_t)(n_base + r) * n + kq, *c1 = c0 + (size_t)16 * n;
        const int k1 = min(n, (z + 1) * slice);
#pragma unroll 8
        for (int k = z * slice; k < k1; k += 16) {
            const bf16x4 a[2] = {*reinterpret_cast<const bf16x4 *>(a0 + k), *reinterpret_cast<const bf16x4 *>(a1 + k)};
            const bf16x4 b[2] = {*reinterpret_cast<const bf16x4 *>(c0 + k), *reinterpret_cast<const bf16x4 *>(c1 + k)};
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[j], acc[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = m_base + 16 * i + kq + v;
                    if (m < M) C[(size_t)m * kHid + n_base + 16 * j + r] = acc[i][j][v];
                }
        return;
    }
    // row sums: the transposed deltas (b1, b2, b3), h3t dy (w4), dy (b4)
    const int row = blockIdx.x - blocks, k = row % kHid, layer = row / kHid;
    const uint16_t *d = (layer == 0 ? tr.d1t : layer == 1 ? tr.d2t : layer == 2 ? tr.d3t : tr.h3t) + (size_t)k * n;
    float s = 0.0f;
    if (layer < 3) {
#pragma unroll 8
        for (int b = threadIdx.x; b < n; b += 256) s += bf2f(d[b]);
    } else if (layer == 3) {
#pragma unroll 8
        for (int b = threadIdx.x; b < n; b += 256) s += bf2f(d[b]) * tr.dy[b];
    } else {
        for (int b = threadIdx.x; b < n; b += 256) s += tr.dy[b];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        g[layer == 0 ? kOffB1 + k : layer == 1 ? kOffB2 + k : layer == 2 ? kOffB3 + k : layer == 3 ? kOffW4 + k : kOffB4] = red[0];
}

// the weight gradients: the slices added in order (of W1, the 8 real input rows)
__global__ __launch_bounds__(256) void k_sum_grads(const float *__restrict__ part, int slices, float *__restrict__ g) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    constexpr int kW = kHid * kHid;
    if (i >= 2 * kW + kIn * kHid) return;
    float s = 0.0f;
#pragma unroll 8
    for (int z = 0; z < slices; ++z) s += part[(size_t)z * kPartial + i];
    g[i < kW ? kOffW3 + i : i < 2 * kW ? kOffW2 + i - kW : kOffW1 + i - 2 * kW] = s;
}

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---------------------------------------------------------------- fused inference
// (the kernel: mlp_infer.h) packed weights: A operands in lane order (W1/4,
// W2 and W3 in bf16), the quartered biases and the output row (bf16-rounded,
// widened)

__global__ void k_pack_fused(const float *__restrict__ p, uint16_t *__restrict__ fw, float *__restrict__ fb) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < kFW1) {
        const int i = idx & 7, lane = (idx >> 3) & 63, ob = idx >> 9;
        const int in = perm_k(lane >> 4, i), out = 16 * ob + (lane & 15);
        fw[idx] = in < kIn ? f2bf(kActScale * p[kOffW1 + in * kHid + out]) : 0;
    }
    if (idx < 2 * kFW2) {
        const int layer = idx / kFW2, r = idx % kFW2;
        const int i = r & 7, lane = (r >> 3) & 63, kb = (r >> 9) & 3, ob = r >> 11;
        const int in = 32 * kb + perm_k(lane >> 4, i), out = 16 * ob + (lane & 15);
        fw[kFW1 + idx] = f2bf(p[(layer ? kOffW3 : kOffW2) + in * kHid + out]);
    }
    if (idx < kFB) {
        float v;
        if (idx < kHid) v = kActScale * p[kOffB1 + idx];
        else if (idx < 2 * kHid) v = kActScale * p[kOffB2 + idx - kHid];
        else if (idx < 3 * kHid) v = kActScale * p[kOffB3 + idx - 2 * kHid];
        else if (idx < 4 * kHid) v = bf2f(f2bf(p[kOffW4 + idx - 3 * kHid]));
        else v = p[kOffB4];
        fb[idx] = v;
    }
}

// samples from an array X[n][8], outputs to y[n]
struct XSource {
    const float *X;
    float *y;
    __device__ uint2 inputs(int64_t p, int g) const {
        const float4 v = *reinterpret_cast<const float4 *>(X + p * kIn + 4 * g);
        return uint2{__builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v.x, v.y}, bf16x2)),
                     __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v.z, v.w}, bf16x2))};
    }
    __device__ int64_t out_base(int64_t p0) const { return p0; }
    __device__ void output(int64_t p0, int i, float v) const { y[p0 + i] = v; }
};

// per-epoch loss: fixed-order sum of the minibatch's partial sums
__global__ void k_loss_add(const double *__restrict__ parts, int nparts, double *__restrict__ loss) {
    double s = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 64) s += parts[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (threadIdx.x == 0) *loss += s;
}

// ---------------------------------------------------------------- host side
struct Net {
    hipStream_t st = nullptr;
    float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;   // [kNParams]
    NetBf16 nb{};
    uint16_t *fw = nullptr;   // fused-inference weights [kFWTotal]
    float *fb = nullptr;      // fused-inference biases and output row [kFB]
    int step = 0;
    // batch workspace
    int cap = 0;
    Transposed tr{};
    float *part = nullptr;    // partial weight gradients [kSplitMax][kPartial]
    double *loss_part = nullptr;
};

static void free_ws(Net &n) {
    for (void *q : {(void *)n.tr.xt, (void *)n.tr.h1t, (void *)n.tr.h2t, (void *)n.tr.h3t, (void *)n.tr.d1t,
                    (void *)n.tr.d2t, (void *)n.tr.d3t, (void *)n.tr.dy, (void *)n.part, (void *)n.loss_part})
        hipFree(q);
    n.tr = Transposed{};
    n.part = nullptr;
    n.loss_part = nullptr;
    n.cap = 0;
}

static hipError_t ensure_ws(Net &n, int cap) {
    if (cap <= n.cap) return hipSuccess;
    free_ws(n);
    hipError_t e;
    const size_t c = (size_t)cap;
#define A(ptr, bytes) if ((e = hipMalloc(&(ptr), (bytes))) != hipSuccess) { free_ws(n); return e; }
    A(n.tr.xt, c * kInPad * 2)
    A(n.tr.h1t, c * kHid * 2) A(n.tr.h2t, c * kHid * 2) A(n.tr.h3t, c * kHid * 2)
    A(n.tr.d1t, c * kHid * 2) A(n.tr.d2t, c * kHid * 2) A(n.tr.d3t, c * kHid * 2)
    A(n.tr.dy, c * 4) A(n.loss_part, (c / kRows) * 8)
    A(n.part, (size_t)kSplitMax * kPartial * 4)
#undef A
    n.cap = cap;
    return hipSuccess;
}

hipError_t net_create(const float *params_host, hipStream_t st, Net **out) {
    Net *n = new Net();
    n->st = st;
    hipError_t e;
    auto bail = [&](hipError_t err) { net_destroy(n); return err; };
    if ((e = hipMalloc(&n->p, kNParams * 4)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->g, kNParams * 4)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->m, kNParams * 4)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->v, kNParams * 4)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->nb.w1t, kHid * kInPad * 2)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->nb.w2t, kHid * kHid * 2)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->nb.w3t, kHid * kHid * 2)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->nb.w2, kHid * kHid * 2)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->nb.w3, kHid * kHid * 2)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->nb.w4, kHid * 2)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->fw, kFWTotal * 2)) != hipSuccess) return bail(e);
    if ((e = hipMalloc(&n->fb, kFB * 4)) != hipSuccess) return bail(e);
    if ((e = hipMemcpyAsync(n->p, params_host, kNParams * 4, hipMemcpyHostToDevice, st)) != hipSuccess) return bail(e);
    if ((e = hipMemsetAsync(n->m, 0, kNParams * 4, st)) != hipSuccess) return bail(e);
    if ((e = hipMemsetAsync(n->v, 0, kNParams * 4, st)) != hipSuccess) return bail(e);
    hipLaunchKernelGGL(k_pack, dim3((kHid * kHid + 255) / 256), dim3(256), 0, st, n->p, n->nb);
    hipLaunchKernelGGL(k_pack_fused, dim3((2 * kFW2 + 255) / 256), dim3(256), 0, st, n->p, n->fw, n->fb);
    if ((e = hipGetLastError()) != hipSuccess) return bail(e);
    // contexts run the network on their own streams: the weights are ready on return
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return bail(e);
    *out = n;
    return hipSuccess;
}

void net_destroy(Net *n) {
    if (!n) return;
    free_ws(*n);
    hipFree(n->p); hipFree(n->g); hipFree(n->m); hipFree(n->v);
    hipFree(n->nb.w1t); hipFree(n->nb.w2t); hipFree(n->nb.w3t); hipFree(n->nb.w2); hipFree(n->nb.w3);
    hipFree(n->nb.w4); hipFree(n->fw); hipFree(n->fb);
    delete n;
}

hipStream_t net_stream(const Net *n) { return n->st; }

hipError_t net_get_params(Net *n, float *host) {
    hipError_t e = hipMemcpyAsync(host, n->p, kNParams * 4, hipMemcpyDeviceToHost, n->st);
    return e == hipSuccess ? hipStreamSynchronize(n->st) : e;
}

static inline unsigned blocks(size_t n) { return (unsigned)((n + 255) / 256); }
// gradients into n.g, after k_train
static hipError_t weight_grads(Net &n, int nb) {
    int slice = 0;
    const int slices = grad_slices(nb, slice);
    hipLaunchKernelGGL(k_weight_grads, dim3(10 * slices + 4 * kHid + 1), dim3(256), 0, n.st, n.tr, nb, slices, slice, n.part,
                       n.g);
    hipLaunchKernelGGL(k_sum_grads, dim3(blocks(2 * kHid * kHid + kIn * kHid)), dim3(256), 0, n.st, n.part, slices, n.g);
    return hipGetLastError();
}

void net_fused_weights(const Net *n, const uint16_t **fw, const float **fb) {
    *fw = n->fw;
    *fb = n->fb;
}

hipError_t net_forward(Net *n, const float *X, int64_t count, float *y, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const int64_t tiles = (count + kFusedTile - 1) / kFusedTile;
    const unsigned grid = (unsigned)std::min<int64_t>(tiles, 256);   // one workgroup per CU
    hipLaunchKernelGGL(k_mlp_infer<XSource>, dim3(grid), dim3(kFusedThreads), 0, st, n->fw, n->fb,
                       XSource{X, y}, count);
    return hipGetLastError();
}

hipError_t net_forward_train(Net *n, const float *X, int count, float *y) {
    if (count <= 0 || count % 16) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_train<Step::outputs>, dim3(count / kRows), dim3(kTrainThreads), 0, n->st, X, n->p, n->nb, count, nullptr,
                       nullptr, 0.0f, y, Transposed{}, nullptr);
    return hipGetLastError();
}

hipError_t net_gradient(Net *n, const float *X, const float *dy, int count, float *grad_host) {
    if (count <= 0 || count % 16) return hipErrorInvalidValue;
    hipError_t e = ensure_ws(*n, count);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_train<Step::gradient>, dim3(count / kRows), dim3(kTrainThreads), 0, n->st, X, n->p, n->nb, count, dy,
                           nullptr, 0.0f, nullptr, n->tr, nullptr);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = weight_grads(*n, count);
    if (e == hipSuccess) e = hipMemcpyAsync(grad_host, n->g, kNParams * 4, hipMemcpyDeviceToHost, n->st);
    if (e == hipSuccess) e = hipStreamSynchronize(n->st);
    return e;
}

// Adam on mean-squared error over minibatches taken in order; the learning
// rate is multiplied by lr_decay after every epoch.  loss_host[epoch] gets
// the epoch's mean loss.
hipError_t net_train(Net *n, const float *X, const float *t, int64_t count, int batch, int epochs, float lr,
                     float lr_decay, double *loss_host) {
    if (batch <= 0 || batch % 16 || count < batch || epochs < 0) return hipErrorInvalidValue;
    hipError_t e = ensure_ws(*n, batch);
    double *loss = nullptr;
    if (e == hipSuccess) e = hipMalloc(&loss, sizeof(double) * std::max(epochs, 1));
    if (e == hipSuccess) e = hipMemsetAsync(loss, 0, sizeof(double) * std::max(epochs, 1), n->st);
    const int64_t n_batches = count / batch;
    const int nparts = batch / kRows;
    for (int ep = 0; ep < epochs && e == hipSuccess; ++ep) {
        for (int64_t bi = 0; bi < n_batches && e == hipSuccess; ++bi) {
            const float *xb = X + bi * batch * kIn;
            const float *tb = t + bi * batch;
            hipLaunchKernelGGL(k_train<Step::train>, dim3(batch / kRows), dim3(kTrainThreads), 0, n->st, xb, n->p, n->nb, batch,
                               nullptr, tb, 1.0f / batch, nullptr, n->tr, n->loss_part);
            hipLaunchKernelGGL(k_loss_add, dim3(1), dim3(64), 0, n->st, n->loss_part, nparts, loss + ep);
            if ((e = weight_grads(*n, batch)) != hipSuccess) break;
            ++n->step;
            const float c1 = 1.0f - powf(0.9f, (float)n->step), c2 = 1.0f - powf(0.999f, (float)n->step);
            hipLaunchKernelGGL(k_adam, dim3(blocks(kNParams)), dim3(256), 0, n->st, n->p, n->g, n->m, n->v, kNParams,
                               lr, 0.9f, 0.999f, 1e-8f, c1, c2);
            hipLaunchKernelGGL(k_pack, dim3((kHid * kHid + 255) / 256), dim3(256), 0, n->st, n->p, n->nb);
            e = hipGetLastError();
        }
        lr *= lr_decay;
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_pack_fused, dim3((2 * kFW2 + 255) / 256), dim3(256), 0, n->st, n->p, n->fw, n->fb);
        e = hipGetLastError();
    }
    std::vector<double> tot(std::max(epochs, 1), 0.0);
    if (e == hipSuccess && epochs > 0)
        e = hipMemcpyAsync(tot.data(), loss, sizeof(double) * epochs, hipMemcpyDeviceToHost, n->st);
    if (e == hipSuccess) e = hipStreamSynchronize(n->st);
    if (e == hipSuccess && loss_host)
        for (int ep = 0; ep < epochs; ++ep) loss_host[ep] = tot[ep] / ((double)n_batches * batch);
    hipFree(loss);
    return e;
}

const int kNetParams = kNParams;

}  // namespace lmo
