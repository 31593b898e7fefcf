// gfx950 kernels for RGBA uint8 image skeletons: fused value stages (noise,
// solarise), mirror as an address remap, 5x5 box blur as a register/DPP
// sliding window, and the histogram/sum reduce side as an LDS epilogue.
//
// Work decomposition.  The paper partitions an image by lines and lets every
// work-group run the whole skeleton tree over its partition, so data passed
// between kernels never leaves the device (Sec. 3.1).  Here one wavefront owns
// a tile = a band of 256 loaded pixels (64 lanes x 4 pixels, one 16-byte load
// per lane per row) by tile_h rows, sweeps it top to bottom, and carries every
// intermediate of the fused stage chain in registers.  A blur band's first and
// last lane only supply halo pixels (248 output pixels per band), so every lane
// loads an aligned group of four pixels and stores four or none; it re-reads 2
// rows above and below its rows.  Halo pixels are recomputed from the input,
// never exchanged.
//
// What bounds it: both sides at once.  The fused MapReduce moves 5.0 TB/s on 8192^2
// and issues VALU operations (42.5 per pixel in the loop, 48 with halo rows and
// epilogue) in 82% of its cycles; an uneven batch, with more halo rows and part
// bands (53 per pixel), in 96%.  1.5 operations per pixel less changed neither
// time measurably; the streams below did.  Streamed
// stores (nt) keep the output out of the memory-side cache: the fused MapReduce
// on 8192^2 133 -> 121 us with streamed loads besides, 4289 x 2847 pointwise
// 4.3 -> 5.4 TB/s.  A streamed store of part of a 128-byte line costs more than it
// saves, so the lanes at a band's ends, whose line the next band shares, store
// normally (8192^2: 136 us with every store streamed, 121 with 8 lanes at each
// end exempt, 139 with 16).
//
// Packed arithmetic.  A pixel is held as two 32-bit registers of u16 pairs,
// e = {R, B} and o = {G, A}.  Noise/solarise use packed 16-bit VALU ops.  Box
// sums stay below 6375 per channel, so packed 32-bit adds never carry between
// the halves and DPP wave shifts fold the neighbour exchange into the adds.
#pragma once
#include "kern_common.h"
#include "kern.h"

#include <algorithm>
#include <type_traits>

namespace skel {

// Noise on one u16 pair: b = two hash bytes; r = b mod 33 computed as
// b - 33 * ((b * 249) >> 13), exact for b in [0, 255]; out = clamp(v + r - 16).
static __device__ __forceinline__ uint32_t noise_half(uint32_t v, uint32_t hb) {
    const u16x2 b = as16(hb);
    const u16x2 q = (b * (u16x2)249) >> (u16x2)13;
    const u16x2 r = b - q * (u16x2)33;
    u16x2 t = as16(v) + r;                                   // v + n + 16 <= 287
    t = __builtin_elementwise_sub_sat(t, (u16x2)16);        // max(v + n, 0)
    t = __builtin_elementwise_min(t, (u16x2)255);
    return as32(t);
}

// Solarise on one u16 pair: min(v, 255 - v) == (v < 128 ? v : 255 - v).
static __device__ __forceinline__ uint32_t sol_half(uint32_t v) {
    const u16x2 t = as16(v);
    return as32(__builtin_elementwise_min(t, (u16x2)255 - t));
}

// Noise followed by solarise on one u16 pair.  With t = v + n, n in [-16, 16],
// solarise(clamp(t, 0, 255)) == max(0, min(t, 255 - t)) for every t in
// [-16, 271]; in unsigned form with t' = t + 16 that is
// min(sat(t' - 16), sat(271 - t')), three packed ops instead of four.
static __device__ __forceinline__ uint32_t noise_sol_half(uint32_t v, uint32_t hb) {
    const u16x2 b = as16(hb);
    const u16x2 q = (b * (u16x2)249) >> (u16x2)13;
    const u16x2 t = as16(v) + (b - q * (u16x2)33);          // t' = v + n + 16 in [0, 287]
    const u16x2 lo = __builtin_elementwise_sub_sat(t, (u16x2)16);
    const u16x2 hi = __builtin_elementwise_sub_sat((u16x2)271, t);
    return as32(__builtin_elementwise_min(lo, hi));
}

// Bytes 1 and 3 of v as a u16 pair (bytes 0 and 2 are v & 0x00FF00FF).
static __device__ __forceinline__ uint32_t odd_bytes(uint32_t v) {
    return __builtin_amdgcn_perm(0u, v, 0x0C030C01u);
}

// h ^ (h >> 16) as one SDWA instruction: the low half becomes lo ^ hi and
// the high half is kept (it is xored with zero).
static __device__ __forceinline__ uint32_t xor_hi_into_lo(uint32_t h) {
    uint32_t r = h;
    asm("v_xor_b32_sdwa %0, %1, %1 dst_sel:WORD_0 dst_unused:UNUSED_PRESERVE src0_sel:WORD_1 src1_sel:WORD_0"
        : "+v"(r)
        : "v"(h));
    return r;
}

// The MurmurHash3 32-bit finaliser (written from its public description) of
// the key seed ^ ((y << 16) | x), x < 2^16.  The key's high half does not
// depend on x, so the finaliser's first xor-shift k ^ (k >> 16) equals
// (S ^ (S >> 16)) ^ x with S = seed ^ (y << 16), a wavefront-uniform value.
static __device__ __forceinline__ uint32_t hash_tail(uint32_t h) {
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    return xor_hi_into_lo(h);
}

// Where a lane's four pixels sit in a row.  xc are their coordinates; with
// `aligned` they are the group ub, ub + 1, .. ub + 3 of an interior band, ub a
// multiple of 4, and stay an aligned group when mirrored (or no stage sees the
// mirrored coordinate).
struct Cols {
    int xc[4];
    int ub;
};

// The hashes of the four pixels.  In an aligned group x = g + j with g a
// multiple of 4, so x ^ s = (g ^ (s & ~3)) + (j ^ (s & 3)) for the row's value s
// and the first product needs one multiplication per lane: the four terms
// (j ^ (s & 3)) c are the row's scalars.
// MODE: the group is known to be aligned, to be looked at pixel by pixel, or
// (ANY_GROUP, an interior lane) aligned unless mirrored in rows of an odd width.
enum { BY_PIXEL = 0, ALIGNED = 1, ANY_GROUP = 2 };
template <int MODE>
static __device__ __forceinline__ void hash4(uint32_t (&h)[4], uint32_t seed, bool fl, const Cols& C, int y, int W) {
    if constexpr (MODE == ANY_GROUP) {
        if (!fl || (W & 3) == 0)
            hash4<ALIGNED>(h, seed, fl, C, y, W);
        else
            hash4<BY_PIXEL>(h, seed, fl, C, y, W);
        return;
    }
    const uint32_t S = seed ^ ((uint32_t)y << 16);
    const uint32_t s = S ^ (S >> 16);
    constexpr uint32_t c = 0x85EBCA6Bu;
    if constexpr (MODE == ALIGNED) {
        const uint32_t g = (uint32_t)(fl ? W - 4 - C.ub : C.ub);
        uint32_t t = (g ^ (s & ~3u)) * c;
        asm("" : "+v"(t));   // keeps the additions below from being folded back into four products
        const uint32_t low = (s & 3u) ^ (fl ? 3u : 0u);
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) h[i] = hash_tail(t + (i ^ low) * c);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) h[i] = hash_tail((s ^ (uint32_t)(fl ? (W - 1 - C.xc[i]) : C.xc[i])) * c);
    }
}

static __device__ __forceinline__ void noise_px(uint32_t& e, uint32_t& o, uint32_t h) {
    e = noise_half(e, h & 0x00FF00FFu);
    o = noise_half(o, odd_bytes(h));
}

static __device__ __forceinline__ void noise_sol_px(uint32_t& e, uint32_t& o, uint32_t h) {
    e = noise_sol_half(e, h & 0x00FF00FFu);
    o = noise_sol_half(o, odd_bytes(h));
}

struct Px4 {
    uint32_t e[4], o[4];
};

template <int MODE>
static __device__ __forceinline__ void noise4(Px4& p, uint32_t seed, bool fl, const Cols& C, int y, int W) {
    uint32_t h[4];
    hash4<MODE>(h, seed, fl, C, y, W);
#pragma unroll
    for (int i = 0; i < 4; ++i) noise_px(p.e[i], p.o[i], h[i]);
}
template <int MODE>
static __device__ __forceinline__ void noise_sol4(Px4& p, uint32_t seed, bool fl, const Cols& C, int y, int W) {
    uint32_t h[4];
    hash4<MODE>(h, seed, fl, C, y, W);
#pragma unroll
    for (int i = 0; i < 4; ++i) noise_sol_px(p.e[i], p.o[i], h[i]);
}
static __device__ __forceinline__ void sol4(Px4& p) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        p.e[i] = sol_half(p.e[i]);
        p.o[i] = sol_half(p.o[i]);
    }
}

// Value stages with a compile-time op sequence (ENC = sum op_k 4^k).
template <int ENC, int K, int MODE>
static __device__ __forceinline__ void apply_const(const OpList& L, Px4& p, const Cols& C, int y, int W) {
    if constexpr (ENC != 0) {
        constexpr int op = ENC & 3;
        if constexpr (op == IOP_NOISE && ((ENC >> 2) & 3) == IOP_SOL) {
            noise_sol4<MODE>(p, L.seed[K], L.flip[K] != 0, C, y, W);
            apply_const<(ENC >> 4), K + 2, MODE>(L, p, C, y, W);
            return;
        } else if constexpr (op == IOP_NOISE) {
            noise4<MODE>(p, L.seed[K], L.flip[K] != 0, C, y, W);
        } else if constexpr (op == IOP_SOL) {
            sol4(p);
        }
        apply_const<(ENC >> 2), K + 1, MODE>(L, p, C, y, W);
    }
}

template <int ENC, int MODE>
static __device__ __forceinline__ void apply_ops(const OpList& L, Px4& p, const Cols& C, int y, int W) {
    if constexpr (ENC == kGeneric) {
        // Stage interpreter: the op list is a kernel argument, so every branch
        // below is uniform across the wavefront.  Codes, flips and seeds are
        // selected from scalar registers: loads from the argument at index k would
        // put a memory latency into every stage of every row.
        uint32_t codes = 0, flips = 0, seed[kMaxOps];
#pragma unroll
        for (int k = 0; k < kMaxOps; ++k) {
            codes |= (uint32_t)(k < L.n ? L.op[k] : 0) << (2 * k);
            flips |= (uint32_t)(L.flip[k] != 0) << k;
            seed[k] = L.seed[k];
        }
        for (int k = 0; codes != 0; ++k, codes >>= 2, flips >>= 1) {
            uint32_t sd = seed[0];
#pragma unroll
            for (int j = 1; j < kMaxOps; ++j) sd = k == j ? seed[j] : sd;
            const uint32_t op = codes & 3u;
            if (op == IOP_NOISE) noise4<MODE>(p, sd, (flips & 1u) != 0, C, y, W);
            if (op == IOP_SOL) sol4(p);
        }
    } else {
        apply_const<ENC, 0, MODE>(L, p, C, y, W);
    }
}

// True when some noise stage sees mirrored coordinates.
static __device__ __forceinline__ bool any_flip(const OpList& L) {
    bool f = false;
#pragma unroll
    for (int k = 0; k < kMaxOps; ++k) f |= k < L.n && L.op[k] == IOP_NOISE && L.flip[k] != 0;
    return f;
}

// floor(s / 25) for each u16 half, s <= 6375: (s * 671089) >> 24 is exact
// there and the product fits 32 bits, so each quotient lands in byte 3 of a
// 24-bit multiply and one byte permute gathers both into a u16 pair.
static __device__ __forceinline__ uint32_t div25_pair(uint32_t s) {
    const uint32_t mlo = (s & 0xFFFFu) * 671089u, mhi = (s >> 16) * 671089u;
    return __builtin_amdgcn_perm(mhi, mlo, 0x0C070C03u);
}

static __device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Input rows in flight per wavefront ahead of the row being computed
// (pointwise chains; a blur keeps one per slot of its ring).
constexpr int kPrefetch = 4;
static_assert(kPrefetch == 4, "pointwise row groups are written out for four slots");
constexpr int kBlurRing = 6;
static_assert(kBlurRing == 6, "blur row groups are written out for six slots");

// Histogram modes: none, or one privatised histogram per work-group with
// kHistWgChan counter words = bins x copies per channel, one copy per class of lanes, so
// that equal values in neighbouring lanes hit different words and banks.  HIST_WG
// (256 bins, 8 copies): counter (c, v, copy) at word c * kHistWgChan + v * copies +
// copy.  HIST_WG128 (128 bins, 16 copies; the chain's last value stage is a
// solarise): at word v * 64 + c * 16 + copy, i.e. byte address v * 256 + c * 64 + 4 *
// copy, which one byte permute builds from the value byte and the lane's copy offset
// (c * 64 is the instruction's offset).
enum { HIST_NONE = 0, HIST_WG = 1, HIST_WG128 = 2 };
constexpr int kHistWgChan = 2048;
constexpr int hist_copies(int hm) { return kHistWgChan / (hm == HIST_WG128 ? 128 : 256); }
// Lanes at either end of a band whose stores are never streamed: 8 x 16 bytes
// cover the 128-byte line that two bands share (see band_tile).
constexpr int kEdgeLanes = 8;
// Kinds of tiles (see band_tile's sweep).
enum { INTERIOR = 0, EDGE_VEC = 1, EDGE_PX = 2 };
constexpr int kByArgs = -1;   // a sweep's cache policy as the arguments give it

// Per-tile geometry and addressing of one image.
struct ImgView {
    const uint8_t* in;
    uint8_t* out;
    int W, H;
    int in_flip, out_flip, write_out;
    int stream;   // STREAM_*
};

// Adds the horizontal 5-sums of the four pixels of each lane to B; lane-1 and
// lane+1 values arrive through DPP wave shifts.  d[-2..5] are the 8 pixels
// around the lane's 4; t1 = d0 + d1, t2 = d2 + d3, and the left neighbour's t2
// is d[-2] + d[-1].  11 operations for 4 pixels (the outer two sums end in a
// three-operand add).  d may hold differences: the packed halves then borrow
// from each other, which cancels in B.
static __device__ __forceinline__ void add_hsum5(const uint32_t (&d)[4], uint32_t (&B)[4]) {
    const uint32_t t1 = d[0] + d[1];
    const uint32_t t2 = d[2] + d[3];
    const uint32_t t12 = t1 + t2;
    // each shifted addend is folded into one DPP add before the last add
    uint32_t s0 = wave_shr1(t2) + t1, s1 = wave_shr1(d[3]) + t12, s2 = wave_shl1(d[0]) + t12, s3 = wave_shl1(t1) + t2;
    asm("" : "+v"(s0), "+v"(s1), "+v"(s2), "+v"(s3));
    B[0] = s0 + d[2] + B[0];
    B[1] += s1;
    B[2] += s2;
    B[3] = s3 + d[1] + B[3];
}

// LITE: the smaller variant of the kernels for the less common chains, with the
// cache policy and the mirror flags read at run time; only the interpreter takes
// images of fewer than 4 columns.
template <int PRE, int POST, bool BLUR, int HM, bool LITE>
static __device__ __forceinline__ void band_tile(const ImgView& V, const OpList& pre, const OpList& post,
                                                 int band, int y0, int y1, int lane, uint32_t* lh) {
    constexpr bool HIST = HM != HIST_NONE;
    const int W = V.W, H = V.H;
    constexpr int bw = BLUR ? kBandOut : kBandPx;
    constexpr int halo = (kBandPx - bw) / 2;
    const int x0 = band * bw;
    const int xend = min(x0 + bw, W);
    const int ub = x0 - halo + lane * 4;
    const bool interior = (x0 - halo >= 0) && (x0 - halo + kBandPx <= W);   // wave-uniform
    const uint32_t nbytes = (uint32_t)W * (uint32_t)H * 4u;
    const __amdgpu_buffer_rsrc_t rin = mk_rsrc(V.in, nbytes);
    const __amdgpu_buffer_rsrc_t rout = mk_rsrc(V.out, nbytes);

    // Histogram addressing: a u16 pair {v0, v1} of HIST_WG shifted left by the
    // counter's size gives both byte offsets in its halves; lane_off is the copy's.
    constexpr int CS = kHistWgChan;
    constexpr uint32_t hsh = HM == HIST_WG128 ? 6 : 5;   // log2 of a counter's bytes over its copies
    const uint32_t lane_off = ((uint32_t)lane & (uint32_t)(hist_copies(HM) - 1)) * 4u;
    static_assert(HM == HIST_NONE || 4 * hist_copies(HM) == 1 << hsh, "copies of a counter are adjacent words");
    char* const lhb = reinterpret_cast<char*>(lh);
    auto count = [&](uint32_t e, uint32_t o, uint32_t inc) {
        if constexpr (HM == HIST_WG128) {
            // byte 1 of the address = the value, byte 0 = the copy offset
            // (< 64), bytes 2-3 = 0; channels R, G, B, A at offsets 0, 64,
            // 128, 192 (e = {R, B}, o = {G, A})
            const uint32_t aR = __builtin_amdgcn_perm(e, lane_off, 0x0C0C0400u);
            const uint32_t aB = __builtin_amdgcn_perm(e, lane_off, 0x0C0C0600u);
            const uint32_t aG = __builtin_amdgcn_perm(o, lane_off, 0x0C0C0400u);
            const uint32_t aA = __builtin_amdgcn_perm(o, lane_off, 0x0C0C0600u);
            atomicAdd(reinterpret_cast<uint32_t*>(lhb + aR), inc);
            atomicAdd(reinterpret_cast<uint32_t*>(lhb + 64 + aG), inc);
            atomicAdd(reinterpret_cast<uint32_t*>(lhb + 128 + aB), inc);
            atomicAdd(reinterpret_cast<uint32_t*>(lhb + 192 + aA), inc);
        } else {
            const uint32_t es = e << hsh, os = o << hsh;
            atomicAdd(reinterpret_cast<uint32_t*>(lhb + 0 * CS * 4 + lane_off + (es & 0xFFFFu)), inc);
            atomicAdd(reinterpret_cast<uint32_t*>(lhb + 1 * CS * 4 + lane_off + (os & 0xFFFFu)), inc);
            atomicAdd(reinterpret_cast<uint32_t*>(lhb + 2 * CS * 4 + lane_off + (es >> 16)), inc);
            atomicAdd(reinterpret_cast<uint32_t*>(lhb + 3 * CS * 4 + lane_off + (os >> 16)), inc);
        }
    };

    // The row sweep, instantiated for interior bands (one 16-byte load and
    // store per lane per row), for bands touching the image edge and for images
    // of fewer than 4 columns.  Prefetched rows stay raw until consumed, so no
    // load result is touched before its row's turn.
    //  EDGE_VEC  a lane loads the 16 bytes nearest to its pixels inside the row
    //            and picks its clamped pixels from them; lanes whose four pixels
    //            are all inside store 16 bytes, the others single pixels.
    //  EDGE_PX   per-pixel loads and stores (a row has no 16 bytes).
    auto sweep = [&](auto kind_tag, auto aligned_tag, auto in_tag, auto out_tag) {
        constexpr int KIND = decltype(kind_tag)::value;
        constexpr bool I = KIND == INTERIOR;
        constexpr int AL = decltype(aligned_tag)::value;
        constexpr int IN = decltype(in_tag)::value, OUT = decltype(out_tag)::value;   // cache policies
        Cols C;
        C.ub = ub;
        int (&xc)[4] = C.xc;
        bool valid[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            xc[i] = I ? (ub + i) : clampi(ub + i, 0, W - 1);
            valid[i] = (ub + i >= x0) && (ub + i < xend);
        }
        // ub and x0 are multiples of 4, so an interior lane is either full or
        // all halo (the first and the last lane of a stencil band)
        const bool full = KIND != EDGE_PX && valid[0] && valid[3];
        // the lanes whose 128-byte line a neighbouring band may write too
        const bool shared_line = lane < halo / 4 + kEdgeLanes || lane >= 64 - halo / 4 - kEdgeLanes;
        uint32_t inc[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) inc[i] = valid[I ? 0 : i] ? 1u : 0u;
        const int mx = V.in_flip ? W - 4 - ub : ub;
        const int vx = I ? mx : clampi(mx, 0, W - 4);
        const uint32_t in_vec = (uint32_t)vx * 4u;
        uint32_t in_px[4];
        int pick[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = V.in_flip ? (W - 1 - xc[i]) : xc[i];
            in_px[i] = (uint32_t)m * 4u;
            pick[i] = m - vx;   // EDGE_VEC: which of the four loaded pixels
        }
        const uint32_t out_vec = (uint32_t)(V.out_flip ? (W - 4 - ub) : ub) * 4u;

        auto load_row = [&](int yy) -> u32x4 {
            const uint32_t rowoff = (uint32_t)yy * (uint32_t)W * 4u;
            if constexpr (KIND != EDGE_PX) {
                if (IN == kByArgs) return V.stream == STREAM_BOTH ? ld128<kStream>(rin, rowoff + in_vec) : ld128(rin, rowoff + in_vec);
                return ld128<IN == kByArgs ? kTemporal : IN>(rin, rowoff + in_vec);
            } else {
                u32x4 r;
                r.x = ld32(rin, rowoff + in_px[0]);
                r.y = ld32(rin, rowoff + in_px[1]);
                r.z = ld32(rin, rowoff + in_px[2]);
                r.w = ld32(rin, rowoff + in_px[3]);
                return r;
            }
        };

        // Pixels of a loaded row in iteration order, split into channel pairs.
        auto unpack = [&](const u32x4& v, Px4& p) {
            uint32_t raw[4];
            if constexpr (KIND == EDGE_VEC) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t lo = pick[i] == 1 ? v.y : v.x, hi = pick[i] == 3 ? v.w : v.z;
                    raw[i] = pick[i] >= 2 ? hi : lo;
                }
            } else if (I && V.in_flip) {
                raw[0] = v.w; raw[1] = v.z; raw[2] = v.y; raw[3] = v.x;
            } else {
                raw[0] = v.x; raw[1] = v.y; raw[2] = v.z; raw[3] = v.w;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                p.e[i] = raw[i] & 0x00FF00FFu;
                p.o[i] = odd_bytes(raw[i]);
            }
        };

        // Final pixels of one output row (e/o = their channel pairs): store
        // (mirrored if out_flip) and count.
        auto emit = [&](const Px4& q, int y) {
            uint32_t fin[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) fin[i] = q.e[i] | (q.o[i] << 8);
            const uint32_t rowoff = (uint32_t)y * (uint32_t)W * 4u;
            if (V.write_out) {
                if (full) {
                    u32x4 v;
                    if (V.out_flip) {
                        v.x = fin[3]; v.y = fin[2]; v.z = fin[1]; v.w = fin[0];
                    } else {
                        v.x = fin[0]; v.y = fin[1]; v.z = fin[2]; v.w = fin[3];
                    }
                    if (OUT == kTemporal || shared_line || (OUT == kByArgs && V.stream == STREAM_NONE))
                        st128(v, rout, rowoff + out_vec);
                    else
                        st128<kStream>(v, rout, rowoff + out_vec);
                } else if constexpr (!I && LITE && PRE != kGeneric) {
                    // The lane that the row ends in: its first one to three pixels are
                    // inside (bands start at multiples of 4).  Offsets and conditions are
                    // formed here: kept over the rows, for either mirror, they were 30
                    // registers, which most of these kernels do not have left.
                    int u = ub;
                    asm("" : "+v"(u));
                    if (u >= x0 && u < xend) {
#pragma unroll
                        for (int i = 0; i < 3; ++i)
                            if (u + i < xend)
                                st32(fin[i], rout, rowoff + (uint32_t)(V.out_flip ? (W - 1 - u - i) : u + i) * 4u);
                    }
                } else if constexpr (!I) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (valid[i]) {
                            const int u = ub + i;
                            st32(fin[i], rout, rowoff + (uint32_t)(V.out_flip ? (W - 1 - u) : u) * 4u);
                        }
                }
            }
            if constexpr (HIST) {
                // Invalid pixels add 0: no branch on per-lane validity.
#pragma unroll
                for (int i = 0; i < 4; ++i) count(q.e[i], q.o[i], inc[i]);
            }
        };

        if constexpr (!BLUR) {
            // Rows are prefetched kPrefetch ahead; slot k is refilled as soon
            // as it is consumed (refills are clamped to the tile, so the last
            // rows re-read cached lines).  Whole groups of kPrefetch rows run
            // in a loop with no early exit and the last y1 - y0 mod kPrefetch
            // rows after it, so the loop back-edge only waits for the oldest
            // row in flight.
            u32x4 nxt[kPrefetch];
#pragma unroll
            for (int d = 0; d < kPrefetch; ++d) nxt[d] = load_row(min(y0 + d, y1 - 1));
            auto row = [&](auto kc, int yy, bool refill) {
                constexpr int k = decltype(kc)::value;
                Px4 p;
                unpack(nxt[k], p);                                              // slot consumed ...
                if (refill) nxt[k] = load_row(min(yy + kPrefetch, y1 - 1));     // ... and refilled
                apply_ops<PRE, AL>(pre, p, C, yy, W);
                emit(p, yy);
            };
            int y = y0;
            for (; y + kPrefetch <= y1; y += kPrefetch) {
                row(std::integral_constant<int, 0>{}, y, true);
                row(std::integral_constant<int, 1>{}, y + 1, true);
                row(std::integral_constant<int, 2>{}, y + 2, true);
                row(std::integral_constant<int, 3>{}, y + 3, true);
            }
            const int rem = y1 - y;
            if (rem > 0) row(std::integral_constant<int, 0>{}, y, false);
            if (rem > 1) row(std::integral_constant<int, 1>{}, y + 1, false);
            if (rem > 2) row(std::integral_constant<int, 2>{}, y + 2, false);
        } else {
            // Sliding 5-row window of pre-blur rows in a ring of 6 slots.  Rows are
            // numbered from y0 - 2, row r in slot r mod 6; output row y0 + t adds
            // row t + 4 and drops row t - 1, so the box sums change by the
            // horizontal sums of the difference of the two: 15 operations for 4
            // pixels and channel pair, where horizontal sums of the entering row,
            // added and later subtracted, took 17.  The sixth slot takes the entering
            // row while the leaving one is still read, so a loop over groups of six
            // rows carries every slot in place (five slots cost 8 register copies a
            // row).  Slots 0-3 start with rows 0-3, slot 5 (row -1) with zeros.
            constexpr int R = kBlurRing;
            uint32_t ringE[R][4], ringO[R][4];
            uint32_t BE[4] = {0, 0, 0, 0}, BO[4] = {0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < 4; ++i) ringE[5][i] = ringO[5][i] = 0;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int rr = clampi(y0 - 2 + s, 0, H - 1);
                Px4 p;
                unpack(load_row(rr), p);
                apply_ops<PRE, AL>(pre, p, C, rr, W);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ringE[s][i] = p.e[i];
                    ringO[s][i] = p.o[i];
                }
                add_hsum5(p.e, BE);
                add_hsum5(p.o, BO);
            }
            // Input rows y+2 ... are prefetched R ahead (one slot per row of
            // an unrolled group, so every slot index is a constant); refills
            // are clamped to the last row the tile needs, y1 + 1.  As above,
            // whole groups of R rows loop with no early exit.
            const int last = min(y1 + 1, H - 1);
            u32x4 nxt[R];
#pragma unroll
            for (int d = 0; d < R; ++d) nxt[d] = load_row(min(y0 + 2 + d, last));
            auto row = [&](auto kc, int yy, bool refill) {
                constexpr int j = decltype(kc)::value;      // (yy - y0) mod R
                constexpr int sn = (j + 4) % R, so = (j + 5) % R;   // slots of the entering and the leaving row
                const int rr = min(yy + 2, H - 1);
                Px4 p;
                unpack(nxt[j], p);                                                // slot consumed ...
                if (refill) nxt[j] = load_row(min(yy + 2 + R, last));             // ... and refilled
                apply_ops<PRE, AL>(pre, p, C, rr, W);
                uint32_t dE[4], dO[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    dE[i] = p.e[i] - ringE[so][i];
                    dO[i] = p.o[i] - ringO[so][i];
                    ringE[sn][i] = p.e[i];
                    ringO[sn][i] = p.o[i];
                }
                add_hsum5(dE, BE);
                add_hsum5(dO, BO);
                Px4 q;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    q.e[i] = div25_pair(BE[i]);
                    q.o[i] = div25_pair(BO[i]);
                }
                apply_ops<POST, AL>(post, q, C, yy, W);
                emit(q, yy);
            };
            int y = y0;
            for (; y + R <= y1; y += R) {
                row(std::integral_constant<int, 0>{}, y, true);
                row(std::integral_constant<int, 1>{}, y + 1, true);
                row(std::integral_constant<int, 2>{}, y + 2, true);
                row(std::integral_constant<int, 3>{}, y + 3, true);
                row(std::integral_constant<int, 4>{}, y + 4, true);
                row(std::integral_constant<int, 5>{}, y + 5, true);
            }
            const int rem = y1 - y;
            if (rem > 0) row(std::integral_constant<int, 0>{}, y, false);
            if (rem > 1) row(std::integral_constant<int, 1>{}, y + 1, false);
            if (rem > 2) row(std::integral_constant<int, 2>{}, y + 2, false);
            if (rem > 3) row(std::integral_constant<int, 3>{}, y + 3, false);
            if (rem > 4) row(std::integral_constant<int, 4>{}, y + 4, false);
        }
    };
    constexpr std::integral_constant<int, kTemporal> keep{};
    constexpr std::integral_constant<int, kStream> stream{};
    constexpr std::integral_constant<int, INTERIOR> inner{};
    constexpr std::integral_constant<int, BY_PIXEL> by_pixel{};
    constexpr std::integral_constant<int, ALIGNED> aligned{};
    if constexpr (LITE) {
        constexpr std::integral_constant<int, kByArgs> by_args{};
        if (PRE == kGeneric && W < 4)
            sweep(std::integral_constant<int, EDGE_PX>{}, by_pixel, keep, keep);
        else if (interior)
            sweep(inner, std::integral_constant<int, ANY_GROUP>{}, by_args, by_args);
        else
            sweep(std::integral_constant<int, EDGE_VEC>{}, by_pixel, keep, keep);
        return;
    } else {
        if (W < 4) {
            sweep(std::integral_constant<int, EDGE_PX>{}, by_pixel, keep, keep);
            return;
        }
        if (!interior) {
            sweep(std::integral_constant<int, EDGE_VEC>{}, by_pixel, keep, keep);
            return;
        }
        if constexpr ((PRE != 0 && PRE != 2) || (POST != 0 && POST != 2)) {   // a noise stage, or unknown
            if ((W & 3) != 0 && (any_flip(pre) || any_flip(post))) {
                sweep(inner, by_pixel, keep, std::integral_constant<int, kByArgs>{});
                return;
            }
        }
        if (V.stream == STREAM_BOTH)
            sweep(inner, aligned, stream, stream);
        else if (V.stream == STREAM_OUT)
            sweep(inner, aligned, keep, stream);
        else
            sweep(inner, aligned, keep, keep);
    }
}

// Zeroes a work-group's histogram, 16 bytes per access.
static __device__ __forceinline__ void clear_hist(uint32_t* lh) {
    u32x4* const q = reinterpret_cast<u32x4*>(lh);
    for (int t = threadIdx.x; t < kHistWgChan; t += blockDim.x) q[t] = u32x4{0, 0, 0, 0};
}

template <int QUAD_PERM>
static __device__ __forceinline__ uint32_t quad_add(uint32_t v) {
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, QUAD_PERM, 0xf, 0xf, true);
}

// Sums the copies of every counter of a privatised LDS histogram and stores the
// counts as one row of 4 x bins words (channel-major) with plain stores.  The
// rows are merged by the histogram finalise kernels, so no device-wide atomics
// are needed.  The counters' copies are adjacent words, 16 (HIST_WG128) or 8: a
// lane reads four of them at once, a wavefront 1 KB without bank conflicts, and
// 4 or 2 neighbouring lanes add up a counter (one word at a time, with a thread
// per counter, clear and row cost a 2048^2 MapReduce 2 us more of 19).  With
// CLEAR every word is zeroed after it is read, leaving the histogram ready for
// the next tile group.  blockDim.x divides 2048.
template <int HM, bool CLEAR = false>
static __device__ __forceinline__ void write_hist_row(uint32_t* lh, uint32_t* row) {
    static_assert(hist_copies(HIST_WG) == 8 && hist_copies(HIST_WG128) == 16, "2 or 4 lanes to a counter");
    u32x4* const q = reinterpret_cast<u32x4*>(lh);
    for (int t = threadIdx.x; t < kHistWgChan; t += blockDim.x) {
        const u32x4 w = q[t];
        if (CLEAR) q[t] = u32x4{0, 0, 0, 0};
        uint32_t n = quad_add<0xB1>((w.x + w.y) + (w.z + w.w));   // + lane ^ 1
        if constexpr (HM == HIST_WG128) {
            n = quad_add<0x4E>(n);                                // + lane ^ 2
            if ((t & 3) == 0) row[((t >> 2) & 3) * 128 + (t >> 4)] = n;
        } else {
            if ((t & 1) == 0) row[(t >> 9) * 256 + ((t & 511) >> 1)] = n;
        }
    }
}

// FL >= 0 fixes the mirror flags at compile time (bit 0: input, bit 1:
// output), which removes the per-row selects of the flipped data order;
// FL = -1 reads them from the arguments (the interpreter and the lite kernels).
// Specialised stencil kernels are held to 128 VGPRs, four wavefronts per SIMD, and
// none keeps anything in private memory: the named chains have a kernel for each
// of the four mirror flags (one reading them took 117-128 registers and, with a
// histogram, up to 68 bytes a lane; mirrored MapReduce of 1125 x 1799 in 64-row tiles
// 49.1 us with it, 44.6 without), and the lite kernels form the offsets of a row's
// last pixels where they are stored (108 bytes a lane before; the same MapReduce of
// noise, blur, solarise 50.1 -> 46.3).
template <int PRE, int POST, bool BLUR, bool HIST, int FL, bool LITE = false>
__global__ void __launch_bounds__(256, BLUR && PRE != kGeneric ? 4 : 1) img_band_kernel(const ImgGroupArgs A) {
    __shared__ __attribute__((aligned(16))) uint32_t lh[HIST ? 4 * kHistWgChan : 1];
    if (A.guard && *A.guard == 0) return;   // a finished while Loop: the whole grid returns
    const int lane = threadIdx.x & 63;
    const int nw = blockDim.x >> 6;
    const int wave = wave_uniform(threadIdx.x >> 6);
    if constexpr (HIST) {
        // Work-group 0 clears the reduce outputs; the merge kernel that runs
        // after this launch adds the work-groups' histogram rows to them.
        if (blockIdx.x == 0) {
            for (int b = threadIdx.x; b < 1024; b += blockDim.x)
                if (A.hist) A.hist[b] = 0;
            if (threadIdx.x < 4 && A.sum) A.sum[threadIdx.x] = 0;
        }
        clear_hist(lh);
        __syncthreads();
    }
    const int tile = blockIdx.x * nw + wave;
    if (tile < A.ntiles) {
        const int band = tile % A.nbands;
        const int chunk = tile / A.nbands;
        const int y0 = chunk * A.tile_h;
        const int y1 = min(y0 + A.tile_h, A.H);
        const ImgView V{A.in, A.out, A.W, A.H, FL < 0 ? A.in_flip : (FL & 1), FL < 0 ? A.out_flip : (FL >> 1),
                        A.write_out, A.stream};
        if (HIST && A.bins == 128)
            band_tile<PRE, POST, BLUR, HIST ? HIST_WG128 : HIST_NONE, LITE>(V, A.pre, A.post, band, y0, y1, lane, lh);
        else
            band_tile<PRE, POST, BLUR, HIST ? HIST_WG : HIST_NONE, LITE>(V, A.pre, A.post, band, y0, y1, lane, lh);
    }
    if constexpr (HIST) {
        __syncthreads();
        uint32_t* const row = A.part + (size_t)blockIdx.x * 4 * A.bins;
        if (A.bins == 128)
            write_hist_row<HIST_WG128>(lh, row);
        else
            write_hist_row<HIST_WG>(lh, row);
    }
}

// A request descriptor read into scalar registers word by word: every lane
// loads the same address, and without the read-back the pointers and sizes
// would stay in vector registers, turning all of the tile's addressing into
// per-lane arithmetic.
static __device__ __forceinline__ BatchReq uniform_req(const BatchReq* p) {
    static_assert(sizeof(BatchReq) % 4 == 0, "descriptor is whole words");
    BatchReq r;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(p);
    uint32_t* dst = reinterpret_cast<uint32_t*>(&r);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(BatchReq) / 4); ++i) dst[i] = (uint32_t)wave_uniform((int)src[i]);
    return r;
}

// Persistent batched kernel: every work-group takes a group of consecutive
// tiles (one per wavefront: adjacent bands of the same rows, so the group
// streams contiguous row segments through one CU's cache, as a work-group of
// the single-image kernel does) from a global ticket counter until the work
// list is exhausted.  The host pads every request's tiles to whole groups, so
// a group never spans two requests: its wavefronts count into one
// work-group histogram, stored as the group's histogram row (row = ticket).
// Each wavefront looks up its tile's request in the tile -> request table;
// padding tiles (past the request's last tile) do nothing.
template <int PRE, int POST, bool BLUR, bool HIST, int FL>
__global__ void __launch_bounds__(256, BLUR && PRE != kGeneric ? 4 : 1) img_batch_kernel(const BatchArgs A) {
    __shared__ __attribute__((aligned(16))) uint32_t lh[HIST ? 4 * kHistWgChan : 1];
    __shared__ uint32_t ticket[2];
    const int lane = threadIdx.x & 63;
    const int wave = wave_uniform(threadIdx.x >> 6);
    const uint32_t nw = blockDim.x >> 6;
    if constexpr (HIST) clear_hist(lh);
    // ticket[] alternates between iterations: thread 0 writes slot i & 1 only
    // after the barrier of iteration i - 1, which every wavefront reaches
    // after reading the same slot in iteration i - 2.  That barrier also
    // orders the previous group's histogram read-and-clear before new counts.
    for (uint32_t it = 0;; ++it) {
        if (threadIdx.x == 0) ticket[it & 1] = atomicAdd(A.counter, 1u);
        __syncthreads();
        const uint32_t g = (uint32_t)wave_uniform((int)ticket[it & 1]);
        if (g * nw >= (uint32_t)A.ntiles) break;   // uniform over the work-group
        const uint32_t t = g * nw + (uint32_t)wave;
        const BatchReq R = uniform_req(A.reqs + wave_uniform((int)A.tile_req[t]));
        const int lt = (int)t - R.tile_begin;
        if (lt < R.nbands * R.nchunks) {
            const int band = lt % R.nbands;
            const int chunk = lt / R.nbands;
            const int y0 = chunk * R.tile_h;
            const int y1 = min(y0 + R.tile_h, R.H);
            const ImgView V{R.in, R.out, R.W, R.H, FL < 0 ? A.in_flip : (FL & 1), FL < 0 ? A.out_flip : (FL >> 1),
                            1, A.stream};
            if (HIST && A.bins == 128)
                band_tile<PRE, POST, BLUR, HIST ? HIST_WG128 : HIST_NONE, PRE == kGeneric>(V, A.pre, A.post, band, y0, y1, lane, lh);
            else
                band_tile<PRE, POST, BLUR, HIST ? HIST_WG : HIST_NONE, PRE == kGeneric>(V, A.pre, A.post, band, y0, y1, lane, lh);
        }
        if constexpr (HIST) {
            __syncthreads();
            uint32_t* const row = A.part + (size_t)g * 4 * A.bins;
            if (A.bins == 128)
                write_hist_row<HIST_WG128, true>(lh, row);
            else
                write_hist_row<HIST_WG, true>(lh, row);
        }
    }
}

// ------------------------------------------------------- instantiations
typedef void (*img_kfn)(const ImgGroupArgs);
typedef void (*batch_kfn)(const BatchArgs);

// A specialised kernel pair (single image, batched).  The instantiations are
// spread over several sources, which compile in parallel.
struct ImgEntry {
    int pre, post;
    bool blur, hist;
    int fl;   // compile-time mirror flags, -1 = from the arguments
    img_kfn fn;
    batch_kfn bfn;
    const char* name;
};

#define SKEL_IMG_ENTRY(P, Q, B, Hh, FL, NAME) \
    {P, Q, B, Hh, FL, img_band_kernel<P, Q, B, Hh, FL, P == kGeneric>, img_batch_kernel<P, Q, B, Hh, FL>, NAME}
// Without a stencil the input is never mirrored (mirrors fold into the
// output address), so those chains need FL 0 and 2 only.
#define SKEL_IMG_POINT(P, Hh, NAME) SKEL_IMG_ENTRY(P, 0, false, Hh, 0, NAME), SKEL_IMG_ENTRY(P, 0, false, Hh, 2, NAME)
#define SKEL_IMG_STENCIL(P, Hh, NAME)                                           \
    SKEL_IMG_ENTRY(P, 0, true, Hh, 0, NAME), SKEL_IMG_ENTRY(P, 0, true, Hh, 1, NAME), \
        SKEL_IMG_ENTRY(P, 0, true, Hh, 2, NAME), SKEL_IMG_ENTRY(P, 0, true, Hh, 3, NAME)

// Chains of up to two value stages on either side of a stencil, or on their own
// (5 = noise twice, 6 = solarise then noise): single images of 4 columns or more.
#define SKEL_IMG_LITE(P, Q, B, Hh, NAME) {P, Q, B, Hh, -1, img_band_kernel<P, Q, B, Hh, -1, true>, nullptr, NAME}
#define SKEL_IMG_LITE_PRE(P, Hh, NAME)                                                          \
    SKEL_IMG_LITE(P, 1, true, Hh, NAME), SKEL_IMG_LITE(P, 2, true, Hh, NAME), SKEL_IMG_LITE(P, 5, true, Hh, NAME), \
        SKEL_IMG_LITE(P, 6, true, Hh, NAME), SKEL_IMG_LITE(P, 9, true, Hh, NAME)

struct ImgEntries {
    const ImgEntry* e;
    int n;
};
ImgEntries img_entries_point();       // no stencil
ImgEntries img_entries_blur();        // stencil
ImgEntries img_entries_blur_hist();   // stencil and histogram
ImgEntries img_entries_generic();     // stage interpreter
ImgEntries img_entries_lite(int k);   // the less common chains, kLiteTables of them
constexpr int kLiteTables = 8;

}  // namespace skel
