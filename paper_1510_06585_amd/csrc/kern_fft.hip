// gfx950 kernels for batched complex fp32 FFT chains (the paper's FFT
// benchmark: FFTs of 512 KiB, i.e. 65536 complex fp32 points, pipelined
// with their inverses, Sec. 4).
//
// A 65536-point transform is computed as 256 x 256 (four-step): with
// n = n1 + 256 n2 and k = k2 + 256 k1,
//   pass A:  for every n1, a 256-point DFT over n2 -> k2, times W_N^(n1 k2),
//            stored transposed as T[k2][n1];
//   pass B:  for every k2, a 256-point DFT over n1 -> k1, giving X[k2 + 256 k1].
// Pass B of one stage and pass A of the next work on the same index (the
// next stage's n1 is this stage's k2), so a fused chain of L stages runs
// L + 1 kernels (A, L - 1 fused "BA", B) instead of 2L: the data between
// two stages never goes back to HBM.
//
// One work-group of 16 COLS threads owns COLS = 32, 16 or 8 columns or rows of one
// transform: it loads a COLS x 256 tile (each row of COLS elements is one run of
// 8 COLS bytes), does the 256-point DFTs in LDS as 16 x 16 (a 16-point DFT per
// thread, a twiddle by W_256, a second 16-point DFT), and stores the tile the
// same way.
// Twiddles come from the 65536 roots of unity computed in double precision on
// the host: W_256^(u p) from a 16 x 16 LDS table in the order the threads read
// it, W_N^(n1 m) as one root per thread times one of a 16 x COLS LDS table.
//
// What bounds it: the three phases of a work-group (load, transform, store) against
// HBM.  Constant element distances carried in scalar offsets and twiddles read from
// tables took the VALU instructions of the three modes from 1457 / 2040 / 884 to
// 1028 / 1709 / 747 with no change in time at 512 transforms.  With streamed results
// and parts of at most kFftRun transforms, whose intermediates then partly stay in the
// memory-side cache, FFT -> IFFT of 512 transforms went from 306 to 288 us, of 256
// from 160 to 144, of 64 from 47.7 to 41.2; in one part it is 318 us at 512.
#include "kern_common.h"
#include "kern.h"

namespace skel {

constexpr int kFftN = kFftPoints;
constexpr int kFftR = 256;     // row / column length
// LDS tile layout: element m of row j at j * kRowStride + m + m / 16.  The
// pad after every 16 elements and the odd row stride keep both the in-row
// stride-16 reads of the DFT and the down-a-column accesses of the loads and
// stores free of bank conflicts (8-byte elements span 2 of the 32 banks).
constexpr int kRowStride = kFftR + kFftR / 16 + 1;
static __device__ __forceinline__ int sx(int j, int m) { return j * kRowStride + m + (m >> 4); }

struct cpx {
    float x, y;
};
static __device__ __forceinline__ cpx cadd(cpx a, cpx b) { return {a.x + b.x, a.y + b.y}; }
static __device__ __forceinline__ cpx csub(cpx a, cpx b) { return {a.x - b.x, a.y - b.y}; }
static __device__ __forceinline__ cpx cmul(cpx a, cpx b) {
    return {__builtin_fmaf(a.x, b.x, -a.y * b.y), __builtin_fmaf(a.x, b.y, a.y * b.x)};
}
// The transform direction DIR is a template parameter: -1 forward
// (W = exp(-2 pi i / N)), +1 inverse, so no twiddle carries a run-time sign.

// a * (DIR * i)
template <int DIR>
static __device__ __forceinline__ cpx cmul_i(cpx a) { return DIR < 0 ? cpx{a.y, -a.x} : cpx{-a.y, a.x}; }

// Roots of unity in LDS, W = exp(2 pi i / N): p16[16 p + u] = W_256^(u p), and for
// the transposed stores row[COLS i + j] = W^(16 n1 i) with n1 = COLS g + j.
template <int COLS>
struct TwLds {
    cpx p16[256], row[16 * COLS];
};

static __device__ __forceinline__ cpx root(const float2* T, uint32_t m) {
    const float2 r = T[m & (uint32_t)(kFftN - 1)];
    return {r.x, r.y};
}

template <bool ROW, int COLS>
static __device__ __forceinline__ void load_tw(TwLds<COLS>& L, const float2* T, int g) {
    const uint32_t t = threadIdx.x;
#pragma unroll
    for (uint32_t i = t; i < 256u; i += 16 * COLS) L.p16[i] = root(T, 256u * (i >> 4) * (i & 15u));
    if (ROW) L.row[t] = root(T, 16u * (t / COLS) * (uint32_t)(COLS * g + t % COLS));
}

template <int DIR>
static __device__ __forceinline__ cpx dir(cpx w) { return {w.x, DIR < 0 ? -w.y : w.y}; }

// Element i of a thread's run: its byte offset in the buffer plus i * STEP.
template <int POLICY = kTemporal>
static __device__ __forceinline__ cpx ld_cpx(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t step) {
    return __builtin_bit_cast(cpx, __builtin_amdgcn_raw_buffer_load_b64(r, off, step, POLICY));
}
template <int POLICY = kTemporal>
static __device__ __forceinline__ void st_cpx(cpx v, __amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t step) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, step, POLICY);
}

// a * W_16^K in direction DIR, the root as a compile-time constant.
template <int DIR, int K>
static __device__ __forceinline__ cpx rot16(cpx a) {
    constexpr float c8 = 0.92387953251128674f, s8 = 0.38268343236508978f, r2 = 0.70710678118654752f;
    constexpr int k = K % 16;
    if constexpr (k == 0) return a;
    else if constexpr (k == 4) return cmul_i<DIR>(a);
    else {
        constexpr float cs[16][2] = {{1, 0},   {c8, s8},   {r2, r2},   {s8, c8},   {0, 1},   {-s8, c8},
                                     {-r2, r2}, {-c8, s8}, {-1, 0},    {-c8, -s8}, {-r2, -r2}, {-s8, -c8},
                                     {0, -1},  {s8, -c8},  {r2, -r2},  {c8, -s8}};
        return cmul(a, cpx{cs[k][0], DIR < 0 ? -cs[k][1] : cs[k][1]});
    }
}

// In-register 4-point DFT of (a, b, c, d).
template <int DIR>
static __device__ __forceinline__ void dft4(cpx& a, cpx& b, cpx& c, cpx& d) {
    const cpx s0 = cadd(a, c), d0 = csub(a, c), s1 = cadd(b, d), d1 = cmul_i<DIR>(csub(b, d));
    a = cadd(s0, s1);
    c = csub(s0, s1);
    b = cadd(d0, d1);
    d = csub(d0, d1);
}

// In-register 16-point DFT, v[c] -> v[k] in natural order, as 4 x 4:
// c = c1 + 4 c2, k = k2 + 4 k1; a 4-point DFT over c2, the twiddle
// W_16^(c1 k2), a 4-point DFT over c1.
template <int DIR, int C1 = 1>
static __device__ __forceinline__ void twiddle16(cpx (&v)[16]) {
    if constexpr (C1 < 4) {
        v[C1 + 4] = rot16<DIR, C1 * 1>(v[C1 + 4]);
        v[C1 + 8] = rot16<DIR, C1 * 2>(v[C1 + 8]);
        v[C1 + 12] = rot16<DIR, C1 * 3>(v[C1 + 12]);
        twiddle16<DIR, C1 + 1>(v);
    }
}

template <int DIR>
static __device__ __forceinline__ void dft16(cpx (&v)[16]) {
#pragma unroll
    for (int c1 = 0; c1 < 4; ++c1) dft4<DIR>(v[c1], v[c1 + 4], v[c1 + 8], v[c1 + 12]);
    // v[c1 + 4 k2] now holds U[c1][k2]
    twiddle16<DIR>(v);
    cpx o[16];
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) {
        cpx a = v[0 + 4 * k2], b = v[1 + 4 * k2], c = v[2 + 4 * k2], d = v[3 + 4 * k2];
        dft4<DIR>(a, b, c, d);
        o[k2] = a;
        o[k2 + 4] = b;
        o[k2 + 8] = c;
        o[k2 + 12] = d;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = o[k];
}

// 256-point DFTs of the COLS rows of a tile, thread t working on row
// j = t / 16 with u = t % 16: on entry v[c] = x[u + 16 c] of row j, on exit
// v[q] = X[u + 16 q].  The input and output element sets of a thread are the
// same, so a second transform of the same rows (the fused pass) starts from
// the registers.  S is the LDS tile used for the transposition in between;
// the call starts with a barrier (other threads may still read S) and ends
// without one.  w[p] = W_256^(u p), p = 1..15.
template <int DIR>
static __device__ __forceinline__ void dft256_reg(cpx* S, const cpx (&w)[16], cpx (&v)[16]) {
    const int j = threadIdx.x >> 4, u = threadIdx.x & 15;
    // m = a + 16 c with a = u: 16-point DFT over c, twiddle W_256^(a p).
    dft16<DIR>(v);
#pragma unroll
    for (int p = 1; p < 16; ++p) v[p] = cmul(v[p], dir<DIR>(w[p]));
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 16; ++p) S[sx(j, 16 * p + u)] = v[p];   // Z[a = u][p] at 16 p + a
    __syncthreads();
    // for p = u: 16-point DFT over a -> k = p + 16 q
#pragma unroll
    for (int a = 0; a < 16; ++a) v[a] = S[sx(j, 16 * u + a)];
    dft16<DIR>(v);
}

static __device__ __forceinline__ void dft256_reg(cpx* S, const cpx (&w)[16], cpx (&v)[16], int d) {
    if (d < 0)
        dft256_reg<-1>(S, w, v);
    else
        dft256_reg<1>(S, w, v);
}

// Twiddle W_N^(n1 k2) (n1 = COLS g + j, k2 = m) and store T[k2][n1].
// A thread stores one column j = t mod COLS at the rows m = m0 + 16 i
// (m0 = t / COLS, i < 16), so its twiddles are a = W^(n1 m0), read once per
// thread, times W^(16 n1 i) from the table that its work-group shares (each a
// root rounded once; forming them per element from two 256-entry tables took
// 9 more operations).
template <int DIR, int COLS>
static __device__ __forceinline__ void store_twiddled(const cpx* S, const TwLds<COLS>& W, cpx a,
                                                      __amdgpu_buffer_rsrc_t out, int g) {
    const int t = threadIdx.x;
    const int j = t % COLS, m0 = t / COLS;
    const uint32_t off = (uint32_t)(m0 * kFftTRow + COLS * g + j) * 8u;
    a = dir<DIR>(a);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const cpx w = i > 0 ? cmul(a, dir<DIR>(W.row[COLS * i + j])) : a;
        st_cpx(cmul(S[sx(j, m0 + 16 * i)], w), out, off, (uint32_t)(16 * i * kFftTRow) * 8u);
    }
}

// MODE 0 (A): in natural order -> T layout; MODE 1 (BA): T -> T (pass B of
// one stage, pass A of the next); MODE 2 (B): T -> natural order.  dir1 is
// the direction of the first DFT, dir2 of the second (MODE 1); scale1 (1/N
// after an inverse stage, else 1) multiplies the result of a stage's pass B.
// The chain's result is stored as a stream.
template <int MODE, int COLS>
__global__ void __launch_bounds__(16 * COLS) fft_pass_kernel(const FftArgs A) {
    __shared__ cpx S[COLS * kRowStride];
    __shared__ TwLds<COLS> W;
    const int b = blockIdx.x / (kFftR / COLS);
    const int g = blockIdx.x % (kFftR / COLS);
    const int t = threadIdx.x;
    // natural order: kFftN elements per transform; transposed (a pass A
    // output, a pass B input): 256 rows of kFftTRow
    constexpr uint32_t kT = kFftR * kFftTRow;
    constexpr uint32_t kIn = MODE == 0 ? kFftN : kT, kOut = MODE == 2 ? kFftN : kT;
    const __amdgpu_buffer_rsrc_t in = mk_rsrc(reinterpret_cast<const cpx*>(A.in) + (size_t)b * kIn, kIn * 8u);
    const __amdgpu_buffer_rsrc_t out = mk_rsrc(reinterpret_cast<cpx*>(A.out) + (size_t)b * kOut, kOut * 8u);
    const int j = t >> 4, u = t & 15;
    const int jc = t % COLS, m0 = t / COLS;   // a thread's column and first row of the tile
    cpx v[16];   // v[c] = element u + 16 c of row j of the tile
    if (MODE == 0) {
        // column n1 = COLS g + j, rows n2 = m: x[n1 + 256 m], staged
        // through LDS (a thread's own elements are 32-byte pieces of 16 rows)
        const uint32_t off = (uint32_t)(COLS * g + jc + kFftR * m0) * 8u;
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = ld_cpx(in, off, (uint32_t)(16 * i * kFftR) * 8u);
    } else {
        // row k2 = COLS g + j of T (T[k2][m] at k2 * kFftTRow + m),
        // straight into registers: for each c the 16 threads of a row read one
        // 128-byte run
        const uint32_t off = (uint32_t)((COLS * g + j) * kFftTRow + u) * 8u;
#pragma unroll
        for (int c = 0; c < 16; ++c) v[c] = ld_cpx(in, off, 128u * c);
    }
    load_tw<MODE != 2, COLS>(W, A.tw, g);
    cpx a{};
    if (MODE != 2) a = root(A.tw, (uint32_t)(COLS * g + jc) * (uint32_t)m0);
    if (MODE == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) S[sx(jc, m0 + 16 * i)] = v[i];
    }
    __syncthreads();
    if (MODE == 0) {
#pragma unroll
        for (int c = 0; c < 16; ++c) v[c] = S[sx(j, u + 16 * c)];
    }
    {
        cpx w[16];
#pragma unroll
        for (int p = 1; p < 16; ++p) w[p] = W.p16[16 * p + u];
        dft256_reg(S, w, v, A.dir1);
        if (MODE == 1) {
            // v[q] = X[k2 + 256 k1] of the first stage at k1 = u + 16 q (k2 =
            // COLS g + j): the second stage's input at n1' = k2, n2' = k1,
            // i.e. exactly what its transform of row j starts from.
            if (A.scale1 != 1.0f)
#pragma unroll
                for (int q = 0; q < 16; ++q) v[q] = {v[q].x * A.scale1, v[q].y * A.scale1};
            dft256_reg(S, w, v, A.dir2);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 16; ++q) S[sx(j, u + 16 * q)] = v[q];
    }
    __syncthreads();
    if (MODE == 0 || MODE == 1) {
        if ((MODE == 0 ? A.dir1 : A.dir2) < 0)
            store_twiddled<-1, COLS>(S, W, a, out, g);
        else
            store_twiddled<1, COLS>(S, W, a, out, g);
    } else {
        // X[k2 + 256 k1] with k2 = COLS g + j, k1 = m
        const uint32_t off = (uint32_t)(COLS * g + jc + kFftR * m0) * 8u;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            cpx x = S[sx(jc, m0 + 16 * i)];
            x = {x.x * A.scale1, x.y * A.scale1};
            const uint32_t step = (uint32_t)(16 * i * kFftR) * 8u;
            if (A.stream != STREAM_NONE)
                st_cpx<kStream>(x, out, off, step);
            else
                st_cpx(x, out, off, step);
        }
    }
}

template <int COLS>
static void fft_launch(const FftArgs& a, int mode, hipStream_t s) {
    void (*const fn)(const FftArgs) =
        mode == 0 ? fft_pass_kernel<0, COLS> : (mode == 1 ? fft_pass_kernel<1, COLS> : fft_pass_kernel<2, COLS>);
    hipLaunchKernelGGL(fn, dim3((unsigned)(a.nfft * (kFftR / COLS))), dim3(16 * COLS), 0, s, a);
}

// Columns per work-group: 32 (256-byte runs, two work-groups per CU), fewer where
// the batch is too small to give every CU one.  FFT -> IFFT, us with 32 / 16 / 8
// columns: 1 transform 18.5 / 14.6 / 12.9, 4: 20.1 / 15.9 / 14.5, 16: 21.7 / 19.5 / 20.2,
// 64: 41.0 / 45.2 / 58.5, 512: 318 / 330 / 437.
int fft_cols(int64_t nfft) { return nfft >= 32 ? 32 : (nfft >= 8 ? 16 : 8); }

hipError_t launch_fft_pass(const FftArgs& a, int mode, hipStream_t s) {
    if (a.nfft <= 0) return hipSuccess;
    if (mode < 0 || mode > 2) return hipErrorInvalidValue;
    switch (fft_cols(a.nfft)) {
        case 32: fft_launch<32>(a, mode, s); break;
        case 16: fft_launch<16>(a, mode, s); break;
        default: fft_launch<8>(a, mode, s); break;
    }
    return hipGetLastError();
}

const char* fft_pass_name(int mode) {
    return mode == 0 ? "fft_pass_a" : (mode == 1 ? "fft_pass_ba" : "fft_pass_b");
}

}  // namespace skel
