// Launch interface between the host runtime (plan/executor) and the gfx950
// kernels.  Plain structs passed by value as kernel arguments.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>

namespace skel {

constexpr int kMaxOps = 8;          // value stages per side of a fused image kernel
constexpr int kBandOut = 248;       // output pixels per wavefront band (stencil kernels)
constexpr int kBandPx = 256;        // pixels a wavefront loads per row (64 lanes x 4)
inline int band_count(int64_t W, bool blur) {
    const int bw = blur ? kBandOut : kBandPx;
    return (int)((W + bw - 1) / bw);
}

// Wavefronts per CU that stencil launches are laid out for: 4 per SIMD, also where
// the registers would let a fifth in, whose tiles are shorter and have more halo
// rows for no more throughput (plain blur, us, tiles for 16 / 20 wavefronts: 8192^2
// 107.9 / 114.2, 2847 x 4289 19.5 / 21.1; persistent batch of 128 709 / 735).
constexpr int kStencilWaves = 16;
// Work-groups with a histogram that fit a CU's LDS: 32 KB each in allocation units of
// 1280 bytes, which the occupancy query (5 groups) leaves out.
constexpr int kHistGroups = 4;

// Value (non-moving) image stages inside a fused kernel.
enum : uint8_t { IOP_NONE = 0, IOP_NOISE = 1, IOP_SOL = 2 };

// A run of value stages.  flip[k] = 1 when stage k sees the mirrored
// coordinate W-1-u of the kernel's iteration coordinate u.
struct OpList {
    int32_t n;
    uint8_t op[kMaxOps];
    uint8_t flip[kMaxOps];
    uint32_t seed[kMaxOps];
};

// Cache policy of a kernel's image streams.  A store marked as a stream does
// not displace other data from the 256 MB memory-side cache, so the input,
// or what the next launch reads, can stay there; marking the loads too pays
// only where the input exceeds that cache anyway.
enum : int32_t { STREAM_NONE = 0, STREAM_OUT = 1, STREAM_BOTH = 2 };
constexpr int64_t kMallBytes = (int64_t)256 << 20;   // memory-side cache
// Policy of a kernel that reads in_bytes: `last` when its output is not to be kept
// for a reader in this plan.  From three quarters of the cache on, little of an input survives
// until a next run could find it there (fp32 chains with 240 MB of input 5.25 ->
// 5.58 TB/s, with 120 MB and one stage 6.7 -> 6.0).
inline int32_t stream_policy(int64_t in_bytes, bool last) {
    return in_bytes >= kMallBytes / 4 * 3 ? STREAM_BOTH : (last ? STREAM_OUT : STREAM_NONE);
}

// Whether a while Loop's images are stored to stay in the memory-side cache for the
// next iteration: a mid-size pair does, a large one does not fit beside the loop's
// input, and a small one is not written faster that way.  Eight iterations of blur5
// with a histogram, us, stored to stay / streamed: 8 MB 140 / 136, 17 MB 162 / 162,
// 30 MB 199 / 205, 67 MB 296 / 334, 144 MB 579 / 551.
inline bool while_keeps(int64_t bytes) { return bytes >= kMallBytes / 12 && bytes < kMallBytes / 8 * 3; }

// One fused image kernel: pre-stages, an optional 5x5 blur, post-stages, an
// optional histogram/sum epilogue.  The kernel iterates over coordinates u of
// the blur's frame (or of its input, without a blur); it reads the input at
// in_flip ? W-1-u : u and writes the output at out_flip ? W-1-u : u.
struct ImgGroupArgs {
    const uint8_t* in;
    uint8_t* out;
    uint32_t* part;      // histogram epilogue: one row of 4 x bins counts per work-group
    uint32_t* hist;      // reduce outputs cleared by work-group 0 (may be null)
    uint64_t* sum;
    int32_t bins;        // values emitted are < bins (128 after a last solarise, else 256)
    int32_t W, H;
    int32_t tile_h;      // rows per tile
    int32_t nbands;      // tiles across a row
    int32_t ntiles;      // nbands * ceil(H / tile_h)
    int32_t in_flip, out_flip;
    int32_t write_out;   // 0 for a reduce-only kernel
    int32_t stream;          // STREAM_*
    const uint32_t* guard;   // while Loop: the launch does nothing when *guard == 0 (null: always runs)
    OpList pre, post;
};

// Compile-time encoding of a value-stage run for specialised kernels:
// sum of op_k * 4^k; -1 selects the generic stage interpreter.
constexpr int kGeneric = -1;
int encode_ops(const OpList& l);

// Launches one fused image kernel with `wg` threads per work-group (64, 128
// or 256).  variant 1 forces the generic interpreter.  *kname receives the
// kernel's name.  t0 / t1 (may be null): events timestamped by the kernel's
// own dispatch (start and end of its execution).
hipError_t launch_img_group(const ImgGroupArgs& a, bool blur, bool hist, int wg, int variant,
                            hipStream_t s, const char** kname, hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr);

const char* img_kernel_name(const ImgGroupArgs& a, bool blur, bool hist, int variant);
// Resident wavefronts per CU of the kernel launch_img_group would pick (16
// when the occupancy query is unavailable, e.g. without a device).
int img_waves_per_cu(const ImgGroupArgs& a, bool blur, bool hist, int wg, int variant);

// Merge of histogram rows (the reduce's merge function, Sec. 3.4): a segment
// owns rows [row_begin, row_begin + nrows) of 4 x bins counts, summed in
// chunks of crows rows by one 1024-thread work-group each, which adds its
// non-zero counts (and the channel sums they imply) to the segment's
// [4][256] histogram (may be null) and [4] sums with device-scope atomics.
// The outputs must be cleared before (hist_zero, or work-group 0 of the image
// kernel that writes the rows).
struct HistSeg {
    uint32_t* hist;
    uint64_t* sum;
    int32_t row_begin, nrows;
    int32_t crows, chunk_begin;
};

// While Loop on the device.  state[0] = 1 while the loop runs, state[1] =
// iterations run, state[2..3] = the previous iteration's tested channel sum
// (uint64), state[4] = chunks of the running merge that are done.  init sets
// {1, 0} and state[4] = 0; step (after each iteration's merge) merges the
// iteration's carried reduce outputs into their accumulators, counts the
// iteration, stores the count to *count_out and clears the flag when
// count == max or the condition fails (kind 0: sum[channel] cmp threshold;
// kind 1: |sum[channel] - previous| cmp threshold, always true after the
// first iteration); copy moves `bytes` from src to dst when max - count is
// odd (the last iteration wrote src).
struct WhileCond {
    int32_t channel, cmp;
    uint64_t threshold;
    int32_t max, kind;
};
// Carried reduce outputs: acc += the iteration's result (null: not carried).
struct WhileMerge {
    const uint32_t* it_hist;
    uint32_t* acc_hist;     // [4][256]
    const uint64_t* it_sum;
    uint64_t* acc_sum;      // [4]
};
struct WhileStep {
    uint32_t* state;         // null: no step
    const uint64_t* sum;     // the iteration's sums
    WhileCond cond;
    WhileMerge merge;
    uint32_t* count_out;
};
struct HistFinArgs {
    const uint32_t* part;
    const uint32_t* guard;   // as ImgGroupArgs::guard
    const HistSeg* segs;   // device array of nseg segments, or null for `one`
    HistSeg one;
    int32_t nseg;
    int32_t nchunks;       // chunks over all segments
    int32_t bins;
    int32_t pad;
    WhileStep step;        // taken by the launch's last chunk to finish
};
// Rows per chunk for rows of 4 x bins words: 8 rows per thread of a
// 1024-thread work-group.
int hist_chunk_rows(int bins);
inline int hist_chunks(int n, int crows) { return n > 0 ? (n + crows - 1) / crows : 0; }
hipError_t launch_hist_merge(const HistFinArgs& a, hipStream_t s);
// Clears every segment's outputs, and *word when given.
hipError_t launch_hist_zero(const HistFinArgs& a, hipStream_t s, uint32_t* word = nullptr);

hipError_t launch_while_init(uint32_t* state, hipStream_t s);
// The step on its own, for an iteration without a merge.
hipError_t launch_while_step(const WhileStep& w, hipStream_t s);
hipError_t launch_while_copy(const uint32_t* state, const void* src, void* dst, uint64_t bytes, uint32_t max,
                             hipStream_t s);

// Work list entry of the batched persistent kernel (one per request).
struct BatchReq {
    const uint8_t* in;
    uint8_t* out;
    uint32_t* hist;
    uint64_t* sum;
    int32_t W, H;
    int32_t nbands, nchunks;
    int32_t tile_begin;  // first global tile index of this request (a multiple of the wavefronts per group)
    int32_t tile_h;      // rows per tile of this request
};
struct BatchArgs {
    const BatchReq* reqs;
    const uint16_t* tile_req;   // request index of every tile
    int32_t nreq;
    int32_t ntiles;
    int32_t has_blur;
    int32_t in_flip, out_flip;
    int32_t has_hist;
    int32_t bins;        // values emitted are < bins
    int32_t stream;      // STREAM_*
    uint32_t* part;      // histogram rows, one per tile group (ticket)
    uint32_t* counter;   // work-queue ticket counter (zeroed before launch)
    OpList pre, post;
};
hipError_t launch_img_batch(const BatchArgs& a, int grid, int wg, hipStream_t s, const char** kname);
// Resident work-groups per CU of the persistent kernel for this chain.
int img_batch_blocks_per_cu(const BatchArgs& a, int wg);

// Fill kernel (graph-safe replacement of memset): n 32-bit words of `value`.
hipError_t launch_fill_u32(void* p, uint64_t nwords, uint32_t value, hipStream_t s);

// ---------------------------------------------------------------- fp32 chains
constexpr int kMaxVecOps = 8;
struct VecGroupArgs {
    const float* in;
    float* out;
    int64_t n;
    int32_t nops;
    int32_t in_flip, out_flip;
    int32_t ept;              // 4-float vectors per thread
    float* partials;          // per work-group partial sums (reduce) or null
    float* sum_out;           // final sum (with partials)
    int32_t write_out;
    int32_t stream;           // STREAM_*
    const float* side[kMaxVecOps];
    float a[kMaxVecOps];
    uint8_t flip[kMaxVecOps];
};
// Launches the chain kernel and, when a.partials is set, the kernel that adds
// the work-group partials into a.sum_out.
hipError_t launch_vec_group(const VecGroupArgs& a, int grid, int wg, hipStream_t s, const char** kname);

// ------------------------------------------------------------ gray volumes
// Fused chain of SEGMENT stages over n voxels (bytes): stage k maps v to
// v < lo[k] ? 0 : (v < hi[k] ? 128 : 255).  in may equal out.
struct GrayArgs {
    const uint8_t* in;
    uint8_t* out;
    int64_t n;
    int32_t nops;
    int32_t ept;          // 16-byte vectors per thread
    int32_t stream;       // STREAM_*
    uint16_t lo[kMaxOps], hi[kMaxOps];   // 0 <= lo <= hi <= 256
};
hipError_t launch_gray_chain(const GrayArgs& a, int grid, int wg, hipStream_t s);

// --------------------------------------------------------------- complex FFT
// Batched 65536-point complex fp32 transforms (interleaved re, im), four-step
// 256 x 256.  mode 0: pass A (natural order in, transposed out), mode 1:
// pass B of a stage fused with pass A of the next, mode 2: pass B
// (transposed in, natural order out).  in and out must not overlap.
struct FftArgs {
    const void* in;
    void* out;
    const float2* tw;    // 65536 roots of unity (cos, sin)(2 pi m / 65536)
    int32_t nfft;        // transforms in the batch
    int32_t dir1, dir2;  // -1 forward, +1 inverse
    float scale1;        // applied to a stage's pass-B result (1/65536 after an inverse)
    int32_t stream;      // STREAM_* of a natural-order result
};
constexpr int kFftPoints = 65536;
// Row stride, in complex elements, of the transposed layout T[k2][n1] that
// passes exchange through plan scratch: 256 + 16 keeps every row on a 128-byte
// line boundary while breaking the power-of-two stride of the column runs.
constexpr int kFftTRow = 256 + 16;
// A batch runs in equal parts of at most kFftRun transforms, each through all
// passes, so that a part's intermediates (0.54 MB a transform, twice) are still
// partly in the memory-side cache when the next pass reads them (FFT -> IFFT, us, one
// part / two: 265 transforms 153 / 163, 285: 175 / 170, 300: 190 / 174, 384: 230 / 216,
// 512: 318 / 288; parts of 128 lose that again to the launches).
constexpr int64_t kFftRun = 280;
// Transforms of a part (the last one may have fewer).
inline int64_t fft_part(int64_t nfft) {
    const int64_t parts = (nfft + kFftRun - 1) / kFftRun;
    return parts > 0 ? (nfft + parts - 1) / parts : 0;
}
int fft_cols(int64_t nfft);   // columns (rows) of a transform per work-group
hipError_t launch_fft_pass(const FftArgs& a, int mode, hipStream_t s);
const char* fft_pass_name(int mode);

// -------------------------------------------------------------------- N-body
struct NBodyArgs {
    const float4* pos_in;   // [N] x,y,z,m
    float4* pos_out;        // [N]
    float4* vel;            // [N] (w unused), updated in place
    float4* acc;            // [N] accelerations (unfused force kernel) or null
    int32_t N;
    int32_t jsplit;         // wavefronts sharing one group of bodies (nbody_group)
    float eps2, G, dt;
    int32_t pad;
};
// Bodies per work-group of the force kernel: 16, 32 or 64.
int nbody_group(int64_t N);
// Fused force + kick-drift (fused = true) or force only into acc.
hipError_t launch_nbody_force(const NBodyArgs& a, bool fused, hipStream_t s, const char** kname);
hipError_t launch_nbody_integrate(const NBodyArgs& a, hipStream_t s, const char** kname);
hipError_t launch_copy_f32x4(const float4* src, float4* dst, int64_t n, hipStream_t s);

// ------------------------------------------------------------------- MLP
hipError_t launch_mlp_forward(const float* params, const float* X, int n, float* y, hipStream_t s);
hipError_t launch_mlp_grad(const float* params, const float* X, const float* t, int n, float* grad,
                           float* loss, float* work, hipStream_t s);
// As launch_mlp_grad over the samples idx[0..n) of X / t (idx may be null).
hipError_t launch_mlp_grad_idx(const float* params, const float* X, const float* t, const int* idx, int n,
                               float* grad, float* loss, float* work, hipStream_t s);
hipError_t launch_mlp_adam(float* params, const float* grad, float* m, float* v, int step, float lr,
                           float b1, float b2, float eps, hipStream_t s);
size_t mlp_grad_work_floats(int n);

}  // namespace skel
