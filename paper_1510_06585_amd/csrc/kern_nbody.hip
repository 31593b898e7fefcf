// gfx950 kernels for the N-body Loop body (Sec. 4 N-Body: direct sum, every
// body reads every position -- the COPY transfer mode of Sec. 3.4).
//
// A work-group owns a group of 16, 32 or 64 bodies and `jsplit` wavefronts;
// wavefront w sums the interactions with the bodies j of its slice of [0, N).
// A lane works on one body; with groups of fewer than 64 bodies, 64 / group
// lanes share a body and take every (64 / group)-th j.  Interactions are
// accumulated in fp32 over the staged j's and added to fp32 running sums; lanes
// and slices are merged in a fixed order.  The fused kernel then applies the
// kick-drift update to its own bodies, so force and integration never
// round-trip through HBM.
//
// What bounds it: VALU issue, 12 full-rate operations and one v_rsq_f32 per
// pair.  A SIMD issues two simple fp32 operations (add, sub, mul, fma) of two
// wavefronts in one 4-cycle slot, but only while every operand is a vector
// register or an inline constant; one scalar operand puts the operation on the
// single full-width port (measured: v_sub_f32 2.25 cycles, with an SGPR operand
// 4.2; v_fma_f32 2.5, v_rsq_f32 10).  So the wavefront stages 64 bodies at a time
// in its own LDS slot (no work-group barrier) and every lane reads them back by
// broadcast into vector registers, where scalar loads of the j stream had
// put three of the thirteen operations on the slow port: 65536 bodies 1450 ->
// 1201 us a step, 44 cycles per pair where these rates would allow 39.
#include "kern_common.h"
#include "kern.h"

namespace skel {

constexpr int kMaxJSplit = 16;
constexpr int kStage = 64;   // bodies a wavefront stages at a time (one per lane)

// LPB lanes work on one body (each takes every LPB-th j of the slice): a
// work-group owns 64 / LPB bodies.  64 VGPRs, so 8 wavefronts per SIMD.
template <bool FUSED, int LPB>
__global__ void __launch_bounds__(64 * kMaxJSplit) nbody_force_kernel(const NBodyArgs A) {
    constexpr int kB = 64 / LPB;
    __shared__ float4 stage[kMaxJSplit][kStage];
    __shared__ float part[kMaxJSplit][3][kB];
    const int l = threadIdx.x & 63, c = l % kB, q = l / kB;
    const int w = wave_uniform(threadIdx.x >> 6);
    const int N = A.N;
    const int i = blockIdx.x * kB + c;
    const float4* __restrict__ P = A.pos_in;
    const float4 pi = P[min(i, N - 1)];
    const int blocks = (N + kStage - 1) / kStage;
    const int per = (blocks + A.jsplit - 1) / A.jsplit;
    const int t0 = w * per, t1 = min(t0 + per, blocks);
    float eps2 = A.eps2;
    asm("" : "+v"(eps2));   // kept in a vector register
    // Lanes past the last body stage a body of mass 0, whose force is 0.
    auto fetch = [&](int t) {
        const int j = t * kStage + l;
        float4 p = P[min(j, N - 1)];
        if (j >= N) p.w = 0.0f;
        return p;
    };
    float4* const S = stage[w];
    float ax = 0.0f, ay = 0.0f, az = 0.0f;
    if (t0 < t1) {
        float4 next = fetch(t0);
        for (int t = t0; t < t1; ++t) {
            wave_lds_sync();
            S[l] = next;
            wave_lds_sync();
            if (t + 1 < t1) next = fetch(t + 1);
            float tx = 0.0f, ty = 0.0f, tz = 0.0f;
#pragma unroll 8
            for (int k = 0; k < kStage / LPB; ++k) {
                const float4 pj = S[k * LPB + q];
                const float dx = pj.x - pi.x;
                const float dy = pj.y - pi.y;
                const float dz = pj.z - pi.z;
                const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
                // d2 >= eps^2 > 0 is never denormal: the bare v_rsq_f32 instruction.
                const float inv = __builtin_amdgcn_rsqf(d2);
                const float s = (pj.w * inv) * (inv * inv);
                tx = __builtin_fmaf(s, dx, tx);
                ty = __builtin_fmaf(s, dy, ty);
                tz = __builtin_fmaf(s, dz, tz);
            }
            ax += tx;
            ay += ty;
            az += tz;
        }
    }
#pragma unroll
    for (int off = kB; off < 64; off <<= 1) {
        ax += __shfl_xor(ax, off, 64);
        ay += __shfl_xor(ay, off, 64);
        az += __shfl_xor(az, off, 64);
    }
    if (q == 0) {
        part[w][0][c] = ax;
        part[w][1][c] = ay;
        part[w][2][c] = az;
    }
    __syncthreads();
    if (w != 0 || q != 0 || i >= N) return;
    float sx = 0.0f, sy = 0.0f, sz = 0.0f;
    for (int k = 0; k < A.jsplit; ++k) {
        sx += part[k][0][c];
        sy += part[k][1][c];
        sz += part[k][2][c];
    }
    sx *= A.G;
    sy *= A.G;
    sz *= A.G;
    if constexpr (FUSED) {
        // kick-drift: v += dt a; r += dt v
        float4 v = A.vel[i];
        v.x = __builtin_fmaf(A.dt, sx, v.x);
        v.y = __builtin_fmaf(A.dt, sy, v.y);
        v.z = __builtin_fmaf(A.dt, sz, v.z);
        A.vel[i] = v;
        float4 r = pi;
        r.x = __builtin_fmaf(A.dt, v.x, r.x);
        r.y = __builtin_fmaf(A.dt, v.y, r.y);
        r.z = __builtin_fmaf(A.dt, v.z, r.z);
        A.pos_out[i] = r;
    } else {
        A.acc[i] = make_float4(sx, sy, sz, 0.0f);
    }
}

__global__ void nbody_integrate_kernel(const NBodyArgs A) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.N) return;
    const float4 a = A.acc[i];
    float4 v = A.vel[i];
    v.x = __builtin_fmaf(A.dt, a.x, v.x);
    v.y = __builtin_fmaf(A.dt, a.y, v.y);
    v.z = __builtin_fmaf(A.dt, a.z, v.z);
    A.vel[i] = v;
    float4 r = A.pos_in[i];
    r.x = __builtin_fmaf(A.dt, v.x, r.x);
    r.y = __builtin_fmaf(A.dt, v.y, r.y);
    r.z = __builtin_fmaf(A.dt, v.z, r.z);
    A.pos_out[i] = r;
}

__global__ void copy_f32x4_kernel(const float4* src, float4* dst, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

// Bodies per work-group: the largest group that still gives 512 work-groups,
// two of 16 wavefronts on every CU (one resident round), else 16.  Measured at
// 16 slices, us a step with groups of 16 / 32 / 64: 1000 bodies 4.2 / 5.6 / 7.8;
// 8192: 24.6 / 25.4 / 44.4; 16384: 84.9 / 83.0 / 85.6; 65536: 1280 / 1216 / 1202.
int nbody_group(int64_t N) { return N >= 64 * 512 ? 64 : (N >= 32 * 512 ? 32 : 16); }

hipError_t launch_nbody_force(const NBodyArgs& a, bool fused, hipStream_t s, const char** kname) {
    if (a.jsplit < 1 || a.jsplit > kMaxJSplit) return hipErrorInvalidValue;
    if (kname) *kname = fused ? "nbody_force_kick_drift" : "nbody_force";
    if (a.N <= 0) return hipSuccess;
    const int group = nbody_group(a.N);
    void (*const fn)(const NBodyArgs) =
        group == 64   ? (fused ? nbody_force_kernel<true, 1> : nbody_force_kernel<false, 1>)
        : group == 32 ? (fused ? nbody_force_kernel<true, 2> : nbody_force_kernel<false, 2>)
                      : (fused ? nbody_force_kernel<true, 4> : nbody_force_kernel<false, 4>);
    hipLaunchKernelGGL(fn, dim3((a.N + group - 1) / group), dim3(64 * a.jsplit), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_nbody_integrate(const NBodyArgs& a, hipStream_t s, const char** kname) {
    if (kname) *kname = "nbody_kick_drift";
    if (a.N <= 0) return hipSuccess;
    hipLaunchKernelGGL(nbody_integrate_kernel, dim3((a.N + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_copy_f32x4(const float4* src, float4* dst, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(copy_f32x4_kernel, dim3((unsigned)blocks), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

}  // namespace skel
