// gfx950 kernels of the cost-model MLP (24 -> 64 -> 64 -> 1, ReLU), the
// learned replacement of the paper's configuration derivation by scattered
// data interpolation (Sec. 3.2).  The layer products run on the matrix cores
// (fp32 MFMA, 16 x 16 x 4), 16 samples at a time:
//  forward   the two hidden layers as 16 x 24 x 64 and 16 x 64 x 64 products,
//            the output unit as a cross-lane dot product;
//  grad      forward, then dh1 = dz2 W2 and the weight gradients
//            dW2 = dz2^T h1 and dW1 = dz1^T x as products over the samples,
//            accumulated over a work-group's groups of 16 and written as one
//            row per work-group;
//  reduce    four threads per parameter add the rows in a fixed order
//            (deterministic, no atomics);
//  adam      one thread per parameter.
//
// What bounds it: latency.  A mini-batch of 256 samples is 16 groups, so a
// group's four 16-unit tiles go to the four wavefronts of a work-group, the
// parameters come in as 16-byte loads all in flight, and rows of 64 units are 68
// words apart in LDS, which lets a lane read four consecutive inputs of a product
// at once and keeps the 16 rows of a read on different banks (64 apart they
// shared one).  Gradient kernel of 256 samples 5.9 us (8.0 with the parameters
// taking a way through private memory, 21.2 with 16 samples per wavefront);
// the rows' sum 4.0 -> 3.0 and 84.7 -> 8.2 (256 rows at most instead of 1024).
// Parameter layout: W1 [64][24], b1 [64], W2 [64][64], b2 [64], W3 [64], b3.
#include "kern_common.h"
#include "kern.h"

#include <algorithm>

namespace skel {

constexpr int kIn = 24, kH1 = 64, kH2 = 64;
constexpr int oW1 = 0, oB1 = oW1 + kH1 * kIn, oW2 = oB1 + kH1, oB2 = oW2 + kH2 * kH1, oW3 = oB2 + kH2,
              oB3 = oW3 + kH2, kNP = oB3 + 1;
static_assert(kNP == 5825, "parameter count");

// Matrix-core formulation.  v_mfma_f32_16x16x4f32 computes D[16x16] +=
// A[16x4] B[4x16] over a wavefront: lane l supplies A[l%16][l/16] and
// B[l/16][l%16] and holds D[4(l/16)+r][l%16] in accumulator register r.  The
// four wavefronts of a work-group share 16 samples and take 16 of a layer's 64
// units each: a 16 x K by K x 16 product of K/4 steps per wavefront and layer.
// Activations are turned from the D layout into the A layout through 16 x 64
// LDS tiles, rows 68 words apart, which the work-group shares.
typedef float f32x4 __attribute__((ext_vector_type(4)));

static __device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int kWaves = 4;
constexpr int kR1 = 28, kR2 = 68;   // row strides of W1 and of 64-unit rows in LDS

struct MlpSmem {
    __attribute__((aligned(16))) float W1[kH1 * kR1];
    __attribute__((aligned(16))) float W2[kH2 * kR2];
    float b1[kH1], b2[kH2], W3[kH2], b3;
};

// Rows of ROW floats, each 16-byte piece one thread's, in two steps: `fetch` only
// issues the loads (a thread past the last piece reads that one again), `store`
// writes LDS.  The pieces stay in registers in between; filled under a predicate
// they went through private memory, one memory latency after another.  The
// source needs 4-byte alignment only.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
template <int ROWS, int ROW, int STRIDE>
struct Rows {
    static constexpr int pieces = ROWS * ROW / 4, per = (pieces + 64 * kWaves - 1) / (64 * kWaves);
    f32x4 v[per];
    __device__ __forceinline__ void fetch(const float* src) {
#pragma unroll
        for (int i = 0; i < per; ++i) {
            const int p = min((int)threadIdx.x + i * 64 * kWaves, pieces - 1);
            v[i] = *reinterpret_cast<const f32x4u*>(src + 4 * p);
        }
    }
    __device__ __forceinline__ void store(float* dst) const {
#pragma unroll
        for (int i = 0; i < per; ++i) {
            const int p = threadIdx.x + i * 64 * kWaves, row = 4 * p / ROW;
            if ((i + 1) * 64 * kWaves <= pieces || p < pieces)   // only a last round is partial
                *reinterpret_cast<f32x4*>(dst + row * STRIDE + (4 * p - row * ROW)) = v[i];
        }
    }
};

struct Params {
    Rows<kH2, kH1, kR2> w2;
    Rows<kH1, kIn, kR1> w1;
    float u, b3;
    __device__ __forceinline__ void fetch(const float* params) {
        const int k = threadIdx.x & 63, q = threadIdx.x >> 6;
        w2.fetch(params + oW2);
        w1.fetch(params + oW1);
        u = params[(q == 0 ? oB1 : (q == 1 ? oB2 : oW3)) + k];
        b3 = params[oB3];
    }
    __device__ __forceinline__ void store(MlpSmem& S) const {
        const int k = threadIdx.x & 63, q = threadIdx.x >> 6;
        w2.store(S.W2);
        w1.store(S.W1);
        if (q < 3) (q == 0 ? S.b1 : (q == 1 ? S.b2 : S.W3))[k] = u;
        if (threadIdx.x == 0) S.b3 = b3;
    }
};

// Products of a 16 x K operand whose rows this lane's c selects (A) with K x 16
// (B), both read as four consecutive k per lane: step (q, j) uses k = 16 q + 4 g + j.
static __device__ __forceinline__ f32x4 dot64(const float* A, const float* B, int g) {
    f32x4 acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 a = *reinterpret_cast<const float4*>(A + 16 * q + 4 * g);
        const float4 b = *reinterpret_cast<const float4*>(B + 16 * q + 4 * g);
        f32x4& d = acc[q & 1];
        d = mfma4(a.x, b.x, d);
        d = mfma4(a.y, b.y, d);
        d = mfma4(a.z, b.z, d);
        d = mfma4(a.w, b.w, d);
    }
    return acc[0] + acc[1];
}

// A row of X as the first layer's operand: features 6 g .. 6 g + 5 of sample `row`,
// zeros unless `in` (the row is read all the same); step s uses k = 6 g + s.
static __device__ __forceinline__ void load_x(const float* X, int row, bool in, int g, float (&xa)[6]) {
    const float* const x = X + (size_t)row * kIn + 6 * g;
    float v[6];
#pragma unroll
    for (int s = 0; s < 6; ++s) v[s] = x[s];
#pragma unroll
    for (int s = 0; s < 6; ++s) xa[s] = in ? v[s] : 0.0f;
}

// Tile t (units 16 t .. 16 t + 15) of the first layer's pre-activations, D
// layout; relu of it goes to H [sample][unit].
static __device__ __forceinline__ f32x4 layer1(const MlpSmem& S, const float (&xa)[6], float* H, int t, int c, int g) {
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < 6; ++s) acc = mfma4(xa[s], S.W1[(16 * t + c) * kR1 + 6 * g + s], acc);
    const float b = S.b1[16 * t + c];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        acc[r] += b;
        H[(4 * g + r) * kR2 + 16 * t + c] = acc[r] > 0.0f ? acc[r] : 0.0f;
    }
    return acc;
}
static __device__ __forceinline__ f32x4 layer2(const MlpSmem& S, const float* H, int t, int c, int g) {
    f32x4 acc = dot64(H + c * kR2, S.W2 + (16 * t + c) * kR2, g);
    const float b = S.b2[16 * t + c];
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] += b;
    return acc;
}
// Sum over the 16 lanes of a row group (fixed butterfly order).
static __device__ __forceinline__ float sum16(float p) {
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) p += __shfl_xor(p, off, 64);
    return p;
}

// A work-group's wavefronts share 16 samples at a time, a tile each (back to back,
// 256 samples 4.1 us and 16384 samples 5.0; 16 samples per wavefront 9.8 and 10.0).
__global__ void __launch_bounds__(64 * kWaves) mlp_forward_kernel(const float* __restrict__ params,
                                                                  const float* __restrict__ X, int n,
                                                                  float* __restrict__ y) {
    __shared__ MlpSmem S;
    __shared__ __attribute__((aligned(16))) float H[16 * kR2];
    __shared__ float Y[kWaves][16];
    const int l = threadIdx.x & 63, c = l & 15, g = l >> 4, w = threadIdx.x >> 6;
    const int groups = (n + 15) / 16;
    float xa[6];
    const auto load = [&](int base) { load_x(X, min(base + c, n - 1), base + c < n, g, xa); };
    Params P;   // in flight together with the first group's samples
    P.fetch(params);
    load(blockIdx.x * 16);
    P.store(S);
    for (int grp = blockIdx.x;;) {
        const int base = grp * 16;
        __syncthreads();   // the parameters; H of the previous group is no longer read
        layer1(S, xa, H, w, c, g);
        __syncthreads();
        const f32x4 z2 = layer2(S, H, w, c, g);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float p = sum16((z2[r] > 0.0f ? z2[r] : 0.0f) * S.W3[16 * w + c]);
            if (c == 0) Y[w][4 * g + r] = p;
        }
        __syncthreads();
        const int s = threadIdx.x;
        if (s < 16 && base + s < n) y[base + s] = ((Y[0][s] + Y[1][s]) + (Y[2][s] + Y[3][s])) + S.b3;
        grp += gridDim.x;
        if (grp >= groups) break;
        load(grp * 16);
    }
}

// Gradient of L = mean over the n samples of (y - t)^2 (X rows idx[b] or b).  A
// work-group takes the groups blockIdx.x, + gridDim.x, ... of 16 samples,
// wavefront w the units 16 w .. 16 w + 15 of both hidden layers, and writes one
// row of kNP + 1 floats (the parameter gradient terms, then the sum of squared
// errors) to part[blockIdx.x].  The rows are summed in order by mlp_grad_reduce.
__global__ void __launch_bounds__(64 * kWaves) mlp_grad_kernel(const float* __restrict__ params,
                                                               const float* __restrict__ X,
                                                               const float* __restrict__ tgt,
                                                               const int* __restrict__ idx, int n,
                                                               float* __restrict__ part) {
    __shared__ MlpSmem S;
    __shared__ __attribute__((aligned(16))) float H[16 * kR2], D[16 * kR2];   // [sample][unit]
    __shared__ float Y[kWaves][16];
    const int l = threadIdx.x & 63, c = l & 15, g = l >> 4, w = threadIdx.x >> 6;
    const int groups = (n + 15) / 16;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 dW2[4] = {zero, zero, zero, zero}, dW1[2] = {zero, zero};
    float gB1 = 0.0f, gB2 = 0.0f, gW3 = 0.0f, gB3 = 0.0f, sq = 0.0f;
    float xa[6], tg[4];
    const auto load = [&](int base) {
        int i = min(base + c, n - 1), b[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) b[r] = min(base + 4 * g + r, n - 1);
        if (idx) {
            i = idx[i];
#pragma unroll
            for (int r = 0; r < 4; ++r) b[r] = idx[b[r]];
        }
        load_x(X, i, base + c < n, g, xa);
#pragma unroll
        for (int r = 0; r < 4; ++r) tg[r] = tgt[b[r]];
    };
    Params P;   // in flight together with the first group's samples
    P.fetch(params);
    load(blockIdx.x * 16);
    P.store(S);
    for (int grp = blockIdx.x;;) {
        const int base = grp * 16;
        __syncthreads();   // the parameters; H and D of the previous group are no longer read
        const f32x4 z1 = layer1(S, xa, H, w, c, g);
        __syncthreads();
        const f32x4 z2 = layer2(S, H, w, c, g);
        const float w3 = S.W3[16 * w + c];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float p = sum16((z2[r] > 0.0f ? z2[r] : 0.0f) * w3);
            if (c == 0) Y[w][4 * g + r] = p;
        }
        __syncthreads();
        // dz2 = dy W3 where z2 > 0 (0 outside the batch)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int s = 4 * g + r;
            const float y = ((Y[0][s] + Y[1][s]) + (Y[2][s] + Y[3][s])) + S.b3;
            const float e = base + s < n ? y - tg[r] : 0.0f;
            const float dy = (2.0f / (float)n) * e;
            const float d = z2[r] > 0.0f ? dy * w3 : 0.0f;
            D[s * kR2 + 16 * w + c] = d;
            gW3 = __builtin_fmaf(dy, z2[r] > 0.0f ? z2[r] : 0.0f, gW3);
            gB2 += d;
            gB3 += dy;
            sq = __builtin_fmaf(e, e, sq);
        }
        __syncthreads();
        // dh1 = dz2 W2 (W2 [o][i]: B[k = o][n = i]); dz1 = dh1 where z1 > 0
        f32x4 dz1 = zero, dz1b = zero;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 a = *reinterpret_cast<const float4*>(D + c * kR2 + 16 * q + 4 * g);
            const float* B = S.W2 + (16 * q + 4 * g) * kR2 + 16 * w + c;
            f32x4& d = q & 1 ? dz1b : dz1;
            d = mfma4(a.x, B[0], d);
            d = mfma4(a.y, B[kR2], d);
            d = mfma4(a.z, B[2 * kR2], d);
            d = mfma4(a.w, B[3 * kR2], d);
        }
        dz1 += dz1b;
        // dW2[o][i] = sum_s dz2[s][o] h1[s][i]: A[m = o][k = s] = D[s][o], B[k = s][n = i] = H[s][i]
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float a = D[(4 * s + g) * kR2 + 16 * w + c];
#pragma unroll
            for (int t = 0; t < 4; ++t) dW2[t] = mfma4(a, H[(4 * s + g) * kR2 + 16 * t + c], dW2[t]);
        }
        __syncthreads();   // every wavefront has read D and H
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float d = z1[r] > 0.0f ? dz1[r] : 0.0f;
            gB1 += d;
            D[(4 * g + r) * kR2 + 16 * w + c] = d;
        }
        if (w == 0)   // the samples' features take h1's place
#pragma unroll
            for (int s = 0; s < 6; ++s) H[c * kR2 + 6 * g + s] = xa[s];
        __syncthreads();
        // dW1[o][k] = sum_s dz1[s][o] x[s][k]: A = D[s][o], B = H[s][k] (k < 24)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float a = D[(4 * s + g) * kR2 + 16 * w + c];
            dW1[0] = mfma4(a, H[(4 * s + g) * kR2 + c], dW1[0]);
            dW1[1] = mfma4(a, c < 8 ? H[(4 * s + g) * kR2 + 16 + c] : 0.0f, dW1[1]);
        }
        grp += gridDim.x;
        if (grp >= groups) break;
        load(grp * 16);
    }
    float* const out = part + (size_t)blockIdx.x * (kNP + 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 16 * w + 4 * g + r;
#pragma unroll
        for (int t = 0; t < 4; ++t) out[oW2 + o * kH1 + 16 * t + c] = dW2[t][r];
        out[oW1 + o * kIn + c] = dW1[0][r];
        if (c < 8) out[oW1 + o * kIn + 16 + c] = dW1[1][r];
    }
    // sums over the 4 row groups (lanes c, c+16, c+32, c+48), fixed order
    for (float* v : {&gB1, &gB2, &gW3, &gB3, &sq}) {
        *v += __shfl_xor(*v, 16, 64);
        *v += __shfl_xor(*v, 32, 64);
    }
    if (g == 0) {
        out[oB1 + 16 * w + c] = gB1;
        out[oB2 + 16 * w + c] = gB2;
        out[oW3 + 16 * w + c] = gW3;
        if (threadIdx.x == 0) {
            out[oB3] = gB3;
            out[kNP] = sq;
        }
    }
}

// grad[p] = sum of the rows' entry p; the loss is the sum of their squared
// errors over n.  Thread (slice, p) of a work-group of 64 parameters adds the rows
// slice, slice + 4, ... in order, eight loads in flight; the slices meet in LDS.
__global__ void __launch_bounds__(256) mlp_grad_reduce_kernel(const float* __restrict__ part, int rows, int n,
                                                              float* __restrict__ grad, float* __restrict__ loss) {
    __shared__ float red[4][64];
    const int k = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int p = min((int)blockIdx.x * 64 + k, kNP);
    float a = 0.0f;
    int r = sl;
    for (; r + 28 < rows; r += 32) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(r + 4 * u) * (kNP + 1) + p];
#pragma unroll
        for (int u = 0; u < 8; ++u) a += v[u];
    }
    float v[7];
#pragma unroll
    for (int u = 0; u < 7; ++u) v[u] = r + 4 * u < rows ? part[(size_t)(r + 4 * u) * (kNP + 1) + p] : 0.0f;
#pragma unroll
    for (int u = 0; u < 7; ++u) a += v[u];
    red[sl][k] = a;
    __syncthreads();
    if (sl != 0 || (int)blockIdx.x * 64 + k > kNP) return;
    const float t = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
    if (p == kNP) {
        if (loss) *loss = t / (float)n;
    } else {
        grad[p] = t;
    }
}

__global__ void mlp_adam_kernel(float* __restrict__ th, const float* __restrict__ g, float* __restrict__ m,
                                float* __restrict__ v, float c1, float c2, float lr, float b1, float b2,
                                float eps) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kNP) return;
    const float gp = g[p];
    const float mp = b1 * m[p] + (1.0f - b1) * gp;
    const float vp = b2 * v[p] + (1.0f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    const float mh = mp / c1, vh = vp / c2;
    th[p] -= lr * mh / (sqrtf(vh) + eps);
}

static int mlp_groups(int n) { return (n + 15) / 16; }
// Gradient rows: a work-group per group of 16 samples, at most one per CU.
static int mlp_rows(int n) { return std::max(1, std::min(256, mlp_groups(n))); }

size_t mlp_grad_work_floats(int n) { return (size_t)mlp_rows(n) * (kNP + 1); }

hipError_t launch_mlp_forward(const float* params, const float* X, int n, float* y, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int wgs = std::min(mlp_groups(n), 1280);   // 5 work-groups' LDS fit a CU
    hipLaunchKernelGGL(mlp_forward_kernel, dim3(wgs), dim3(64 * kWaves), 0, s, params, X, n, y);
    return hipGetLastError();
}

hipError_t launch_mlp_grad_idx(const float* params, const float* X, const float* t, const int* idx, int n,
                               float* grad, float* loss, float* work, hipStream_t s) {
    if (n <= 0) return hipErrorInvalidValue;
    const int rows = mlp_rows(n);
    hipLaunchKernelGGL(mlp_grad_kernel, dim3(rows), dim3(64 * kWaves), 0, s, params, X, t, idx, n, work);
    hipLaunchKernelGGL(mlp_grad_reduce_kernel, dim3((kNP + 1 + 63) / 64), dim3(256), 0, s, (const float*)work, rows,
                       n, grad, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(const float* params, const float* X, const float* t, int n, float* grad, float* loss,
                           float* work, hipStream_t s) {
    return launch_mlp_grad_idx(params, X, t, nullptr, n, grad, loss, work, s);
}

hipError_t launch_mlp_adam(float* params, const float* grad, float* m, float* v, int step, float lr, float b1,
                           float b2, float eps, hipStream_t s) {
    // Bias corrections 1 - beta^t in double, rounded once: for beta2 = 0.999
    // and small t the difference cancels, and rounding beta^t to fp32 before
    // subtracting would cost ~1.5e-5 relative in 1 - beta2^2.
    const float c1 = (float)(1.0 - pow((double)b1, (double)step));
    const float c2 = (float)(1.0 - pow((double)b2, (double)step));
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((kNP + 255) / 256), dim3(256), 0, s, params, grad, m, v, c1, c2, lr,
                       b1, b2, eps);
    return hipGetLastError();
}

}  // namespace skel
