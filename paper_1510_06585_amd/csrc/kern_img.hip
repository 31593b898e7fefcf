// Image runtime: the reduce side's merge kernels, the while Loop's control
// kernels, and the dispatch of the fused image kernels (kern_img_dev.h).
#include <hip/hip_ext.h>

#include "kern_img_dev.h"

namespace skel {

static __device__ __forceinline__ u32x4 ldg128(const uint32_t* p) { return *reinterpret_cast<const u32x4*>(p); }

static __device__ __forceinline__ int seg_of(const HistFinArgs& F, int chunk) {
    if (!F.segs) return 0;
    int lo = 0, hi = F.nseg - 1;
    while (lo < hi) {   // last segment with chunk_begin <= chunk
        const int mid = (lo + hi + 1) >> 1;
        if (F.segs[mid].chunk_begin <= chunk) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Sum of rows [0, nrows) (stride `words`) of `base` by a 1024-thread work-
// group: thread (g, q), g < G = 4096 / words, sums the 16-byte word group q of
// rows g, g + G, ... with kSumUnroll loads in flight, and the G partial sums
// of q meet in LDS.  Threads with g == 0 return the total of their q.
constexpr int kFinThreads = 1024;
constexpr int kSumUnroll = 8;
static __device__ __forceinline__ u32x4 sum_rows(const uint32_t* base, int nrows, int words, u32x4* red) {
    const int nq = words >> 2;
    const int G = kFinThreads / nq;
    const int q = threadIdx.x % nq, g = threadIdx.x / nq;
    u32x4 acc[kSumUnroll];
#pragma unroll
    for (int u = 0; u < kSumUnroll; ++u) acc[u] = u32x4{0, 0, 0, 0};
    for (int r0 = g; r0 < nrows; r0 += kSumUnroll * G) {
        u32x4 v[kSumUnroll];
#pragma unroll
        for (int u = 0; u < kSumUnroll; ++u) {
            const int r = r0 + u * G;
            v[u] = r < nrows ? ldg128(base + (size_t)r * words + 4 * q) : u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int u = 0; u < kSumUnroll; ++u) acc[u] += v[u];
    }
#pragma unroll
    for (int u = 1; u < kSumUnroll; ++u) acc[0] += acc[u];
    __syncthreads();   // red may still be read by a previous call
    red[threadIdx.x] = acc[0];
    __syncthreads();
    u32x4 t = u32x4{0, 0, 0, 0};
    if (g == 0)
        for (int k = 0; k < G; ++k) t += red[k * nq + q];
    return t;
}

// A value of the iteration's results.  SHARED: other work-groups of this launch
// added to it with device-scope atomics.
template <bool SHARED, typename T>
static __device__ __forceinline__ T ld_result(const T* p) {
    return SHARED ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}

// One step of a while Loop by the whole work-group; the loop is running.
template <bool SHARED>
static __device__ __forceinline__ void while_step(const WhileStep& S) {
    const WhileMerge& M = S.merge;
    const WhileCond& c = S.cond;
    uint32_t* const st = S.state;
    if (M.acc_hist)
        for (int b = threadIdx.x; b < 1024; b += blockDim.x) M.acc_hist[b] += ld_result<SHARED>(M.it_hist + b);
    if (M.acc_sum && threadIdx.x < 4) M.acc_sum[threadIdx.x] += ld_result<SHARED>(M.it_sum + threadIdx.x);
    if (threadIdx.x != 0) return;
    const uint32_t n = st[1] + 1u;
    st[1] = n;
    *S.count_out = n;
    uint64_t* prev = reinterpret_cast<uint64_t*>(st + 2);
    const uint64_t s = ld_result<SHARED>(S.sum + c.channel);
    bool go = true;
    uint64_t v = s;
    if (c.kind == 1) {
        v = s >= *prev ? s - *prev : *prev - s;
        *prev = s;
    }
    if (c.kind == 0 || n > 1u) {
        switch (c.cmp) {
            case 0: go = v > c.threshold; break;
            case 1: go = v >= c.threshold; break;
            case 2: go = v < c.threshold; break;
            default: go = v <= c.threshold; break;
        }
    }
    if (!go || n >= (uint32_t)c.max) st[0] = 0u;
}

// Merge (one launch after the kernels that wrote the rows): work-group k sums
// the rows of chunk k.  A segment of one chunk gets its outputs written with
// plain stores; the chunks of a longer segment add their non-zero counts, and
// the channel sums they imply, to its outputs with device-scope atomics, the
// outputs having been cleared before the rows were written (by
// hist_zero_kernel or by work-group 0 of the image kernel).
__global__ void __launch_bounds__(kFinThreads) hist_merge_kernel(const HistFinArgs F) {
    __shared__ u32x4 red[kFinThreads];
    __shared__ unsigned long long csum[4];
    __shared__ bool last_chunk;
    if (F.guard && *F.guard == 0) return;
    const int k = blockIdx.x;
    const HistSeg& S = F.segs ? F.segs[seg_of(F, k)] : F.one;
    const int words = 4 * F.bins;
    const int r0 = S.row_begin + (k - S.chunk_begin) * S.crows;
    const int r1 = min(r0 + S.crows, S.row_begin + S.nrows);
    const bool direct = S.nrows <= S.crows;
    if (threadIdx.x < 4) csum[threadIdx.x] = 0;
    const u32x4 n = sum_rows(F.part + (size_t)r0 * words, max(r1 - r0, 0), words, red);
    if ((int)threadIdx.x < (words >> 2)) {
        const int b = 4 * threadIdx.x;
        const int c = b >> __builtin_ctz((unsigned)F.bins), v = b & (F.bins - 1);
        if (S.hist) {
            uint32_t* h = S.hist + c * 256 + v;
            if (direct) {
                *reinterpret_cast<u32x4*>(h) = n;
            } else {
                if (n.x) atomicAdd(h, n.x);
                if (n.y) atomicAdd(h + 1, n.y);
                if (n.z) atomicAdd(h + 2, n.z);
                if (n.w) atomicAdd(h + 3, n.w);
            }
        }
        const unsigned long long t = (unsigned long long)v * n.x + (unsigned long long)(v + 1) * n.y +
                                     (unsigned long long)(v + 2) * n.z + (unsigned long long)(v + 3) * n.w;
        if (t) atomicAdd(&csum[c], t);
    }
    const int per = 256 - F.bins;
    if (direct && S.hist && (int)threadIdx.x < per) {   // bins above `bins`: 4 x per zero words
        const int b = 4 * threadIdx.x;
        const int c = b / per, v = F.bins + b % per;
        *reinterpret_cast<u32x4*>(S.hist + c * 256 + v) = u32x4{0, 0, 0, 0};
    }
    __syncthreads();
    if (threadIdx.x < 4 && S.sum) {
        if (direct)
            S.sum[threadIdx.x] = csum[threadIdx.x];
        else if (csum[threadIdx.x])
            atomicAdd((unsigned long long*)&S.sum[threadIdx.x], csum[threadIdx.x]);
    }
    if (F.step.state == nullptr) return;
    // A while Loop's step needs every chunk's result: the last chunk to finish
    // takes it.  What it reads of other work-groups was added by device-scope
    // atomics, which are performed before their wave's counter drops and which
    // device-scope loads see, so the ticket needs no cache write-back (a
    // __threadfence in every chunk made the iteration 3 us longer than a launch
    // of its own).  Every work-group has read the guard before its ticket, so
    // clearing the flag here stops later launches only.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) last_chunk = atomicAdd(&F.step.state[4], 1u) + 1u == gridDim.x;
    __syncthreads();
    if (!last_chunk) return;
    if (threadIdx.x == 0) F.step.state[4] = 0u;
    if (direct)
        while_step<false>(F.step);
    else
        while_step<true>(F.step);
}

// Clears the histogram and sums of every segment (one work-group each), and *word.
__global__ void hist_zero_kernel(const HistFinArgs F, uint32_t* word) {
    if (F.guard && *F.guard == 0) return;
    if (word && blockIdx.x == 0 && threadIdx.x == 0) *word = 0;
    const HistSeg& S = F.segs ? F.segs[blockIdx.x] : F.one;
    for (int b = threadIdx.x; b < 1024; b += blockDim.x)
        if (S.hist) S.hist[b] = 0;
    if (threadIdx.x < 4 && S.sum) S.sum[threadIdx.x] = 0;
}

__global__ void while_init_kernel(uint32_t* st) {
    if (threadIdx.x == 0) {
        st[0] = 1u;
        st[1] = 0u;
        st[4] = 0u;
    }
}

constexpr int kStepThreads = 256;
__global__ void __launch_bounds__(kStepThreads) while_step_kernel(const WhileStep S) {
    const uint32_t running = S.state[0];
    __syncthreads();   // every thread has read the flag before thread 0 may clear it
    if (running != 0u) while_step<false>(S);
}

// Copies src to dst (nvec 16-byte vectors, then 4-byte words up to `words`)
// when max - (iterations run) is odd: the last iteration then wrote src.
__global__ void while_copy_kernel(const uint32_t* st, const uint32_t* src, uint32_t* dst, uint64_t words,
                                  uint64_t nvec, uint32_t max) {
    if ((max - st[1]) % 2u == 0u) return;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += stride)
        reinterpret_cast<u32x4*>(dst)[i] = reinterpret_cast<const u32x4*>(src)[i];
    for (uint64_t i = nvec * 4 + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride)
        dst[i] = src[i];
}

__global__ void fill_u32_kernel(uint32_t* p, uint64_t n, uint32_t v) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// ------------------------------------------------------------------ host side
int encode_ops(const OpList& l) {
    int e = 0, m = 1;
    for (int k = 0; k < l.n; ++k) {
        e += m * (int)l.op[k];
        m *= 4;
    }
    return e;
}

ImgEntries img_lite_0();
ImgEntries img_lite_1();
ImgEntries img_lite_2();
ImgEntries img_lite_3();
ImgEntries img_lite_4();
ImgEntries img_lite_5();
ImgEntries img_lite_6();
ImgEntries img_lite_7();

ImgEntries img_entries_lite(int k) {
    ImgEntries (*const f[kLiteTables])() = {img_lite_0, img_lite_1, img_lite_2, img_lite_3,
                                            img_lite_4, img_lite_5, img_lite_6, img_lite_7};
    return f[k]();
}

// The kernels of a chain: one specialised for it and its mirror flags, else a lite
// one (run-time flags; single images of 4 columns or more only, W = 0: a batch),
// else the interpreter.
static const ImgEntry* find_entry(const OpList& pre, const OpList& post, bool blur, bool hist, int in_flip,
                                  int out_flip, int variant, int W) {
    const int pe = encode_ops(pre), qe = encode_ops(post);
    const int fl = (in_flip ? 1 : 0) | (out_flip ? 2 : 0);
    if (variant == 0 && pre.n <= 6 && post.n <= 6) {
        const auto find = [&](const ImgEntries& t, int f) -> const ImgEntry* {
            for (int i = 0; i < t.n; ++i) {
                const ImgEntry& e = t.e[i];
                if (e.pre == pe && e.post == qe && e.blur == blur && e.hist == hist && e.fl == f) return &e;
            }
            return nullptr;
        };
        const ImgEntries t = !blur ? img_entries_point() : (hist ? img_entries_blur_hist() : img_entries_blur());
        if (const ImgEntry* e = find(t, fl)) return e;
        if (W >= 4)
            for (int k = 0; k < kLiteTables; ++k)
                if (const ImgEntry* e = find(img_entries_lite(k), -1)) return e;
    }
    const ImgEntries g = img_entries_generic();
    for (int i = 0; i < g.n; ++i)
        if (g.e[i].blur == blur && g.e[i].hist == hist) return &g.e[i];
    return nullptr;
}

int img_waves_per_cu(const ImgGroupArgs& a, bool blur, bool hist, int wg, int variant) {
    const ImgEntry* e = find_entry(a.pre, a.post, blur, hist, a.in_flip, a.out_flip, variant, a.W);
    int nb = 0;
    if (!e || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(e->fn), wg, 0) !=
                  hipSuccess ||
        nb <= 0) {
        (void)hipGetLastError();
        return 16;
    }
    return nb * (wg / 64);
}

const char* img_kernel_name(const ImgGroupArgs& a, bool blur, bool hist, int variant) {
    const ImgEntry* e = find_entry(a.pre, a.post, blur, hist, a.in_flip, a.out_flip, variant, a.W);
    return e ? e->name : "";
}

hipError_t launch_img_group(const ImgGroupArgs& a, bool blur, bool hist, int wg, int variant, hipStream_t s,
                            const char** kname, hipEvent_t t0, hipEvent_t t1) {
    const ImgEntry* e = find_entry(a.pre, a.post, blur, hist, a.in_flip, a.out_flip, variant, a.W);
    if (!e) return hipErrorInvalidValue;
    if (kname) *kname = e->name;
    if (a.ntiles <= 0) {
        // nothing to launch: the requested events still mark this point
        hipError_t r = t0 ? hipEventRecord(t0, s) : hipSuccess;
        if (r == hipSuccess && t1) r = hipEventRecord(t1, s);
        return r;
    }
    const int waves = wg / 64;
    const int grid = (a.ntiles + waves - 1) / waves;
    if (t0 || t1) {
        // the events take their timestamps from the kernel's own dispatch,
        // so they bracket its execution and nothing else
        ImgGroupArgs arg = a;
        void* args[] = {&arg};
        return hipExtLaunchKernel(reinterpret_cast<const void*>(e->fn), dim3(grid), dim3(wg), args, 0, s, t0, t1,
                                  0);
    }
    hipLaunchKernelGGL(e->fn, dim3(grid), dim3(wg), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_img_batch(const BatchArgs& a, int grid, int wg, hipStream_t s, const char** kname) {
    const ImgEntry* e = find_entry(a.pre, a.post, a.has_blur != 0, a.has_hist != 0, a.in_flip, a.out_flip, 0, 0);
    if (!e) return hipErrorInvalidValue;
    if (kname) *kname = e->name;
    if (wg != 256 && wg != 128 && wg != 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(e->bfn, dim3(grid), dim3(wg), 0, s, a);
    return hipGetLastError();
}

int hist_chunk_rows(int bins) { return kSumUnroll * (kFinThreads / bins); }

static bool valid_step(const WhileStep& w) {
    return w.state && w.cond.channel >= 0 && w.cond.channel <= 3 && w.cond.kind >= 0 && w.cond.kind <= 1 &&
           !w.merge.acc_hist == !w.merge.it_hist && !w.merge.acc_sum == !w.merge.it_sum;
}

hipError_t launch_hist_merge(const HistFinArgs& a, hipStream_t s) {
    if (a.bins != 128 && a.bins != 256) return hipErrorInvalidValue;
    if (a.nchunks <= 0) return hipSuccess;
    if (a.step.state && !valid_step(a.step)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(hist_merge_kernel, dim3(a.nchunks), dim3(kFinThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_hist_zero(const HistFinArgs& a, hipStream_t s, uint32_t* word) {
    if (a.nseg <= 0) return hipSuccess;
    hipLaunchKernelGGL(hist_zero_kernel, dim3(a.nseg), dim3(256), 0, s, a, word);
    return hipGetLastError();
}

int img_batch_blocks_per_cu(const BatchArgs& a, int wg) {
    const ImgEntry* e = find_entry(a.pre, a.post, a.has_blur != 0, a.has_hist != 0, a.in_flip, a.out_flip, 0, 0);
    if (!e) return 0;
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(e->bfn), wg, 0) != hipSuccess)
        return 0;
    return nb;
}

hipError_t launch_while_init(uint32_t* state, hipStream_t s) {
    hipLaunchKernelGGL(while_init_kernel, dim3(1), dim3(64), 0, s, state);
    return hipGetLastError();
}

hipError_t launch_while_step(const WhileStep& w, hipStream_t s) {
    if (!valid_step(w)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(while_step_kernel, dim3(1), dim3(kStepThreads), 0, s, w);
    return hipGetLastError();
}

hipError_t launch_while_copy(const uint32_t* state, const void* src, void* dst, uint64_t bytes, uint32_t max,
                             hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (bytes % 4) return hipErrorInvalidValue;
    const uint64_t words = bytes / 4;
    const bool aligned = (((uintptr_t)src | (uintptr_t)dst) & 15u) == 0;
    const uint64_t nvec = aligned ? words / 4 : 0;
    uint64_t blocks = ((aligned ? nvec : words) + 255) / 256;
    blocks = std::max<uint64_t>(1, std::min<uint64_t>(blocks, 8192));
    hipLaunchKernelGGL(while_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s, state, (const uint32_t*)src,
                       (uint32_t*)dst, words, nvec, max);
    return hipGetLastError();
}

hipError_t launch_fill_u32(void* p, uint64_t nwords, uint32_t value, hipStream_t s) {
    if (nwords == 0) return hipSuccess;
    uint64_t blocks = (nwords + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t*)p, nwords, value);
    return hipGetLastError();
}

}  // namespace skel
