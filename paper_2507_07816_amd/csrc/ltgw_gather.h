// Device code shared by the statistic kernels (ltgw_kernels.hip) and the
// stack kernels of the learned proposer (ltgw_stack.hip): the gather from a
// stored spectrogram, the per-segment accumulation, the results, the XCD
// order of workgroups and the in-band segment windows.
#pragma once
#include "ltgw_internal.h"

#pragma clang fp contract(off)

namespace ltgw {

extern "C" __device__ float ltgw_sbuf_f32(__amdgpu_buffer_rsrc_t, int vindex, int voffset,
                                          int soffset, int aux)
    __asm("llvm.amdgcn.struct.ptr.buffer.load.f32");
extern "C" __device__ unsigned short ltgw_sbuf_u16(__amdgpu_buffer_rsrc_t, int vindex, int voffset,
                                                   int soffset, int aux)
    __asm("llvm.amdgcn.struct.ptr.buffer.load.i16");
extern "C" __device__ unsigned char ltgw_sbuf_u8(__amdgpu_buffer_rsrc_t, int vindex, int voffset,
                                                 int soffset, int aux)
    __asm("llvm.amdgcn.struct.ptr.buffer.load.i8");

// Word 3 of a gfx9 buffer resource: 32-bit data format, no swizzle.
constexpr int kBufDword3 = 0x00020000;

template <int STORE>
struct Store;
template <>
struct Store<LTGW_STORE_F32> {
    static constexpr int kBytes = 4;
    // the element as an FP32 value whose sign is the count bit
    __device__ static float load(__amdgpu_buffer_rsrc_t r, int i, int soff) { return ltgw_sbuf_f32(r, i, 0, soff, 0); }
    // returns |value| and adds the count bit
    __device__ static float get(__amdgpu_buffer_rsrc_t r, int i, int soff, int &cnt) {
        float p = ltgw_sbuf_f32(r, i, 0, soff, 0);
        cnt += (int)(__float_as_uint(p) >> 31);
        return __builtin_fabsf(p);
    }
};
template <>
struct Store<LTGW_STORE_BF16> {
    static constexpr int kBytes = 2;
    __device__ static float load(__amdgpu_buffer_rsrc_t r, int i, int soff) {
        return __uint_as_float((unsigned)ltgw_sbuf_u16(r, i, 0, soff, 0) << 16);
    }
    __device__ static float get(__amdgpu_buffer_rsrc_t r, int i, int soff, int &cnt) {
        unsigned u = ltgw_sbuf_u16(r, i, 0, soff, 0);
        cnt += (int)(u >> 15);
        return __builtin_fabsf(__uint_as_float(u << 16));
    }
};
template <>
struct Store<LTGW_STORE_FP8> {
    static constexpr int kBytes = 1;
    __device__ static float load(__amdgpu_buffer_rsrc_t r, int i, int soff) {
        return __builtin_amdgcn_cvt_f32_fp8((int)ltgw_sbuf_u8(r, i, 0, soff, 0), 0);
    }
    __device__ static float get(__amdgpu_buffer_rsrc_t r, int i, int soff, int &cnt) {
        unsigned u = ltgw_sbuf_u8(r, i, 0, soff, 0);
        cnt += (int)(u >> 7);
        return __builtin_fabsf(__builtin_amdgcn_cvt_f32_fp8((int)u, 0));
    }
};

template <>
struct Store<kStoreCoarse> {
    static constexpr int kBytes = 4;
    // the upper half is the bfloat16 power sum, the low byte the count
    __device__ static float get(__amdgpu_buffer_rsrc_t r, int i, int soff, int &cnt) {
        const unsigned u = __float_as_uint(ltgw_sbuf_f32(r, i, 0, soff, 0));
        cnt += (int)(u & 0xffu);
        return __uint_as_float(u & 0xffff0000u);
    }
};

// An element every lane of the wavefront reads at the same address, through
// the constant address space: for arrays no kernel writes while it runs,
// this makes the read a scalar load.
template <typename T>
__device__ inline T uniform_load(const T *p, int64_t i) {
    return ((const __attribute__((address_space(4))) T *)p)[i];
}

// ---------------------------------------------------------------------------
// Statistic (Sec. 2).  A lane carries TPL templates (f0 256 apart, so each
// of them is a coalesced wavefront access); segments go in batches of U so
// that U*TPL independent gathers are in flight per wavefront.  FP32 partial
// sums over chunks of 32 segments are carried in FP64.
constexpr int kChunk = 32;

// Bin-scaled track factor H_j of one (detector, group): from a table, or
// formed on the fly as RN(RN(g_j D_j) T_sft) (batched searches, whose sky
// patches would make a full table too large).  Both are wavefront-uniform.
struct HTable {
    const double *H;
    __device__ double operator()(int j) const { return H[j]; }
    __device__ double lane(int j) const { return H[j]; }  // j differs from lane to lane
};
struct HFromGD {
    const double *g;  // [n_seg] of the group's (n, tau)
    const double *D;  // [n_seg] of the group's sky direction
    double t_sft;
    __device__ double operator()(int j) const {
        const double h = uniform_load(g, j) * uniform_load(D, j);
        return h * t_sft;
    }
    __device__ double lane(int j) const {
        const double h = g[j] * D[j];
        return h * t_sft;
    }
};

template <int TPL>
struct Acc {
    double s[TPL], w1[TPL], w2[TPL];
    int cnt[TPL], nin[TPL];
    __device__ void zero() {
        for (int t = 0; t < TPL; ++t) {
            s[t] = w1[t] = w2[t] = 0.0;
            cnt[t] = nin[t] = 0;
        }
    }
};

// SHIFT = 1 reads a 2x2-coarsened store (pairs of segments and of bins; the
// caller passes cshift + 1 and the pair's first-segment track factor): the
// coarse column of fine column b is b >> 1, i.e. index trunc(v) >> 1.
template <int STORE, bool MOMENTS, int TPL, int U, class HS, int SHIFT = 0>
__device__ __forceinline__ void seg_batch(const DetView &D, __amdgpu_buffer_rsrc_t rs, const HS &hs,
                                          int j, const double (&f0)[TPL], float (&sc)[TPL],
                                          float (&w1c)[TPL], float (&w2c)[TPL], Acc<TPL> &acc) {
    const unsigned nb = (unsigned)D.n_bins;
    double h[U];
#pragma unroll
    for (int k = 0; k < U; ++k) h[k] = hs(j + k);
    unsigned idx[TPL][U];
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const double x = f0[t] * h[k];
            const double vv = x + D.cshift;
            // a negative index wraps to a large unsigned value: out of range, reads 0
            idx[t][k] = (unsigned)__double2int_rz(vv) >> SHIFT;
        }
    float p[TPL][U];
#pragma unroll
    for (int k = 0; k < U; ++k)
#pragma unroll
        for (int t = 0; t < TPL; ++t)
            p[t][k] = Store<STORE>::get(rs, (int)idx[t][k], (j + k) * D.pitch_bytes, acc.cnt[t]);
    // the weights are read unconditionally (wave-uniform loads, selected per
    // lane): a load guarded by the lane's in-band test would become a branch
    float wv[U];
    if (MOMENTS) {
#pragma unroll
        for (int k = 0; k < U; ++k) wv[k] = uniform_load(D.w, j + k);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const float wq = uniform_load(D.wq, j + k);
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            sc[t] = __builtin_fmaf(wq, p[t][k], sc[t]);
            if (MOMENTS) {
                const bool inb = (idx[t][k] - 1u) < nb;
                acc.nin[t] += inb ? 1 : 0;
                const float wj = inb ? wv[k] : 0.0f;
                w1c[t] += wj;
                w2c[t] = __builtin_fmaf(wj, wj, w2c[t]);
            }
        }
    }
}

// Moments in the loop cost as much as the statistic: a test, a select, two sums and a
// count per evaluation.  Where every f0 of the wavefront is in band in every segment of
// a chunk, and that is most chunks, the chunk adds 32 segments and the same two weight
// sums to all of them, so those come from here: lane l forms the sums of chunk
// first + l step, segment by segment like a template's, for 64 chunks at a time.
// (80 groups of 4000 f0 over 5400 FP8 segments: 690 us before, 535 in eval_kernel and
// 444 with the segments shared.)
struct ChunkWeights {
    float w1 = 0.0f, w2 = 0.0f;
    int first = 0, step = 1, have = 0;
    __device__ __forceinline__ void load(const float *w, int c, int by, int n_full) {
        first = c;
        step = by;
        have = 64;
        w1 = w2 = 0.0f;
        const int mine = c + (int)(threadIdx.x & 63) * by;
        if (mine < n_full)
#pragma unroll 8
            for (int k = 0; k < kChunk; ++k) {
                const float x = w[mine * kChunk + k];
                w1 += x;
                w2 = __builtin_fmaf(x, x, w2);
            }
    }
    // chunk c of those first, first + by, ..
    __device__ __forceinline__ void get(const float *w, int c, int by, int n_full, float &u1, float &u2) {
        int l = have ? (c - first) / step : 64;
        if (l >= 64) {
            load(w, c, by, n_full);
            l = 0;
        }
        u1 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w1), l));
        u2 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w2), l));
    }
};

__device__ __forceinline__ double read_lane(double x, int l) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint64_t lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, l);
    const uint64_t hi = (unsigned)__builtin_amdgcn_readlane((int)(u >> 32), l);
    return __builtin_bit_cast(double, hi << 32 | lo);
}

// Whether all of the wavefront's f0 (f0[t] ascending over the lanes) are in band in all
// segments of the whole chunk from j: the column is monotone in f0.  A lane looks at
// segment j + lane % 32.
template <int TPL, class HS>
__device__ __forceinline__ bool chunk_in_band(const DetView &D, const HS &hs, int j, const double (&f0)[TPL]) {
    const double h = hs.lane(j + (int)(threadIdx.x & (kChunk - 1)));
    bool in = true;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const double xa = read_lane(f0[t], 0) * h, xb = read_lane(f0[t], 63) * h;
        in = in && __double2int_rz(xa + D.cshift) >= 1 && __double2int_rz(xb + D.cshift) <= D.n_bins;
    }
    return __all(in);
}

// All segments of one detector.
// Segments [jb, je) of detector D to visit for the runs [blk0, blk1) of 64 f0
// of group grp: the in-band window widened to whole chunks (chunks outside
// add exact zeros, so skipping them leaves every sum bit-identical); all
// segments when D has no windows.  Wave-uniform.
__device__ __forceinline__ void seg_window(const DetView &D, int grp, int blk0, int blk1, int &jb, int &je) {
    jb = 0;
    je = D.n_seg;
    if (!D.win) return;
    int lo = D.n_seg, hi = -1;
    const int end = blk1 < D.win_blocks ? blk1 : D.win_blocks;
    for (int b = blk0; b < end; ++b) {
        const int2 w = D.win[(int64_t)grp * D.win_blocks + b];
        lo = min(lo, w.x);
        hi = max(hi, w.y);
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
    if (hi < lo) {
        je = 0;
        return;
    }
    jb = (lo / kChunk) * kChunk;
    je = min(D.n_seg, (hi / kChunk + 1) * kChunk);
}

template <int STORE, bool MOMENTS, int TPL, int U, class HS, int SHIFT = 0>
__device__ __forceinline__ void accumulate_det(const DetView &D, const HS &hs,
                                               const double (&f0)[TPL], Acc<TPL> &acc, int jb = 0,
                                               int je = -1) {
    if (je < 0) je = D.n_seg;
    // one resource per detector, n_bins + 2 records (a row with its guards);
    // the row is the instruction's scalar byte offset
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)D.store, Store<STORE>::kBytes, D.n_bins + 2, kBufDword3);
    int j = jb;
    ChunkWeights cw;
    for (; j + kChunk <= je; j += kChunk) {
        float sc[TPL], w1c[TPL], w2c[TPL];
        for (int t = 0; t < TPL; ++t) sc[t] = w1c[t] = w2c[t] = 0.0f;
        if (MOMENTS && chunk_in_band<TPL>(D, hs, j, f0)) {
#pragma unroll 1
            for (int b = 0; b < kChunk; b += U)
                seg_batch<STORE, false, TPL, U, HS, SHIFT>(D, rs, hs, j + b, f0, sc, w1c, w2c, acc);
            float u1, u2;
            cw.get(D.w, j / kChunk, 1, D.n_seg / kChunk, u1, u2);
            for (int t = 0; t < TPL; ++t) {
                w1c[t] = u1;
                w2c[t] = u2;
                acc.nin[t] += kChunk;
            }
        } else {
#pragma unroll 1
            for (int b = 0; b < kChunk; b += U)
                seg_batch<STORE, MOMENTS, TPL, U, HS, SHIFT>(D, rs, hs, j + b, f0, sc, w1c, w2c, acc);
        }
        for (int t = 0; t < TPL; ++t) {
            acc.s[t] += (double)sc[t];
            if (MOMENTS) {
                acc.w1[t] += (double)w1c[t];
                acc.w2[t] += (double)w2c[t];
            }
        }
    }
    if (j < je) {
        float sc[TPL], w1c[TPL], w2c[TPL];
        for (int t = 0; t < TPL; ++t) sc[t] = w1c[t] = w2c[t] = 0.0f;
        for (; j < je; ++j)
            seg_batch<STORE, MOMENTS, TPL, 1, HS, SHIFT>(D, rs, hs, j, f0, sc, w1c, w2c, acc);
        for (int t = 0; t < TPL; ++t) {
            acc.s[t] += (double)sc[t];
            if (MOMENTS) {
                acc.w1[t] += (double)w1c[t];
                acc.w2[t] += (double)w2c[t];
            }
        }
    }
}

// Segments [jb, je) (whole chunks, but for the detector's last) shared by the W
// wavefronts of a workgroup, a chunk each in turn: its counts stay with its wavefront,
// its sums go to LDS and the first wavefront adds them in chunk order, so the sums are
// those of accumulate_det bit for bit.  b: the LDS buffer to use next.
template <bool MOMENTS, int TPL, int W>
struct SharedSums {
    float s[2][MOMENTS ? 3 : 1][TPL][W][64];
};

template <int STORE, bool MOMENTS, int TPL, int U, int W, class HS>
__device__ __forceinline__ void accumulate_shared(const DetView &D, const HS &hs, const double (&f0)[TPL], Acc<TPL> &acc,
                                                  int jb, int je, int wv, SharedSums<MOMENTS, TPL, W> &part, int &b) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)D.store, Store<STORE>::kBytes, D.n_bins + 2, kBufDword3);
    const int lane = (int)threadIdx.x & 63, chunks = (je + kChunk - 1) / kChunk;
    ChunkWeights cw;
    for (int c0 = jb / kChunk; c0 < chunks; c0 += W, b ^= 1) {
        int j = (c0 + wv) * kChunk;
        const int jc = min(j + kChunk, je);
        float sc[TPL], w1c[TPL], w2c[TPL];
        for (int t = 0; t < TPL; ++t) sc[t] = w1c[t] = w2c[t] = 0.0f;
        if (MOMENTS && jc - j == kChunk && chunk_in_band<TPL>(D, hs, j, f0)) {
            float u1, u2;
            cw.get(D.w, c0 + wv, W, D.n_seg / kChunk, u1, u2);
            for (int t = 0; t < TPL; ++t) {
                w1c[t] = u1;
                w2c[t] = u2;
                acc.nin[t] += kChunk;
            }
#pragma unroll 1
            for (; j < jc; j += U) seg_batch<STORE, false, TPL, U>(D, rs, hs, j, f0, sc, w1c, w2c, acc);
        }
#pragma unroll 1
        for (; j + U <= jc; j += U) seg_batch<STORE, MOMENTS, TPL, U>(D, rs, hs, j, f0, sc, w1c, w2c, acc);
#pragma unroll 1
        for (; j < jc; ++j) seg_batch<STORE, MOMENTS, TPL, 1>(D, rs, hs, j, f0, sc, w1c, w2c, acc);
        for (int t = 0; t < TPL; ++t) {
            part.s[b][0][t][wv][lane] = sc[t];
            if constexpr (MOMENTS) {
                part.s[b][1][t][wv][lane] = w1c[t];
                part.s[b][2][t][wv][lane] = w2c[t];
            }
        }
        __syncthreads();  // the other buffer's sums were read before it
        if (wv == 0)
            for (int k = 0; k < min(W, chunks - c0); ++k)
                for (int t = 0; t < TPL; ++t) {
                    acc.s[t] += (double)part.s[b][0][t][k][lane];
                    if constexpr (MOMENTS) {
                        acc.w1[t] += (double)part.s[b][1][t][k][lane];
                        acc.w2[t] += (double)part.s[b][2][t][k][lane];
                    }
                }
    }
}

// The wavefronts' counts added up in the first one.
template <bool MOMENTS, int TPL, int W>
__device__ __forceinline__ void add_counts(Acc<TPL> &acc, int wv, int (&count)[MOMENTS ? 2 : 1][TPL][W][64]) {
    const int lane = (int)threadIdx.x & 63;
    for (int t = 0; t < TPL; ++t) {
        count[0][t][wv][lane] = acc.cnt[t];
        if constexpr (MOMENTS) count[1][t][wv][lane] = acc.nin[t];
    }
    __syncthreads();
    if (wv == 0)
        for (int k = 1; k < W; ++k)
            for (int t = 0; t < TPL; ++t) {
                acc.cnt[t] += count[0][t][k][lane];
                if constexpr (MOMENTS) acc.nin[t] += count[1][t][k][lane];
            }
}

// Results of a lane's templates; template index grp*n_f0 + i.
template <bool MOMENTS, int TPL>
__device__ __forceinline__ void store_results(const Acc<TPL> &acc, const int (&i)[TPL], int grp,
                                              int n_f0, double *s, int32_t *c, int32_t *n,
                                              double *w1, double *w2, float *out_s, int32_t *out_c,
                                              int32_t *out_n, unsigned long long *in_band_total) {
    if (MOMENTS) {
        // in-band total for the roofline's algorithmic bytes (one atomic per wave)
        unsigned long long nw = 0;
        for (int t = 0; t < TPL; ++t) nw += (i[t] < n_f0) ? (unsigned long long)acc.nin[t] : 0ull;
        for (int o = 32; o > 0; o >>= 1) nw += __shfl_xor(nw, o, 64);
        if (in_band_total) atomicAdd(in_band_total, (threadIdx.x & 63) == 0 ? nw : 0ull);
    }
    for (int t = 0; t < TPL; ++t) {
        if (i[t] >= n_f0) continue;
        const int64_t q = (int64_t)grp * n_f0 + i[t];
        s[q] = acc.s[t];
        c[q] = acc.cnt[t];
        if (out_s) out_s[q] = (float)acc.s[t];
        if (out_c) out_c[q] = acc.cnt[t];
        if (MOMENTS) {
            n[q] = acc.nin[t];
            w1[q] = acc.w1[t];
            w2[q] = acc.w2[t];
            if (out_n) out_n[q] = acc.nin[t];
        }
    }
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Block w runs on XCD w % 8; it is given the (f0 tile, group) pair
// number start(x) + w / 8 in tile-major order (group fastest), where XCD x
// owns a contiguous range of pairs.  So the blocks resident on one XCD at a
// time cover one f0 tile of many neighbouring (tau, n, sky) groups: their
// tracks start at the same bins and stay close for similar tau and n, so
// their reads of each row overlap in that XCD's L2.  (Group-major order, one
// group's successive f0 tiles side by side, reads disjoint bins and measured
// slower.)
// A launch may cover a slice [first, first + gridDim.x) of the pairs (a
// generation of the grid); the XCD ranges are taken within the slice.
constexpr int kXcds = 8;
__device__ inline void xcd_tile_group(int w, int n_blocks, int n_tiles, int &tile, int &grp,
                                      int first = 0, int total = -1) {
    const int x = w % kXcds, k = w / kXcds;
    const int base = n_blocks / kXcds, extra = n_blocks % kXcds;
    const int start = x * base + (x < extra ? x : extra);
    const int p = first + start + k;
    const int n_groups = (total < 0 ? n_blocks : total) / n_tiles;
    tile = p / n_groups;
    grp = p % n_groups;
}

// A value that is the same in every lane, moved to scalar registers word by
// word (lets the compiler treat descriptors read from memory as uniform).
template <class T>
__device__ __forceinline__ T uniform(const T &x) {
    static_assert(sizeof(T) % 4 == 0, "whole words only");
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
    for (unsigned k = 0; k < sizeof(T) / 4; ++k) w[k] = __builtin_amdgcn_readfirstlane(w[k]);
    T y;
    __builtin_memcpy(&y, w, sizeof(T));
    return y;
}

}  // namespace ltgw
