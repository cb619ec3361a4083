// Data preparation (Sec. 2): strain -> Hann-windowed short Fourier transforms
// -> normalised power rho = P ln 2 / (running median of P over frequency).
//
// Segment j is samples [j N, (j + 1) N) of the strain.  Per chunk of segments:
//   the powers P_k = |X_k|^2 of the band and its median halo, for the lengths that a
//   workgroup can hold from one kernel that reads the strain and writes them
//   (ltgw_fft.hip); for the others a batched real-to-complex FFT (hipFFT, FP32) of the
//   raw segments, and the Hann window applied in frequency: with the periodic
//   window w_n = 1/2 - 1/2 cos(2 pi n / N) = 1/2 - e^{2 pi i n/N}/4 - e^{-2 pi i n/N}/4
//   the windowed transform is X_k/2 - (X_{k-1} + X_{k+1})/4 (X_{-1} = conj X_1 and
//   X_{N/2+1} = conj X_{N/2-1} for real input);
//   normalise_kernel: each bin's median, the (h + 1)-th smallest of its window of
//   2 h + 1 powers, and the ratio.  Under Gaussian noise P_k is exponential with
//   mean S_k and median S_k ln 2, hence rho_k = P_k ln 2 / median.
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <cmath>
#include <cstdio>
#include <vector>

#include "ltgw_ctx.h"
#include "ltgw_fft.h"
#include "median_slide.h"

#pragma clang fp contract(off)

namespace ltgw {

constexpr int kSftMaxWindow = 257;

__device__ __forceinline__ float2 spec_at(const float2 *row, int64_t k, int64_t half) {
    // X_{-1} = conj X_1, X_{half+1} = conj X_{half-1} (real input)
    if (k < 0) {
        const float2 z = row[-k];
        return make_float2(z.x, -z.y);
    }
    if (k > half) {
        const float2 z = row[2 * half - k];
        return make_float2(z.x, -z.y);
    }
    return row[k];
}

// |windowed transform|^2 of bin k from a row of the raw transform
__device__ __forceinline__ float hann_power(const float2 *row, int64_t k, int64_t half) {
    const float2 z = row[k], zm = spec_at(row, k - 1, half), zp = spec_at(row, k + 1, half);
    const float re = 0.5f * z.x - 0.25f * (zm.x + zp.x);
    const float im = 0.5f * z.y - 0.25f * (zm.y + zp.y);
    const float a = re * re;
    const float b = im * im;
    return a + b;
}

// the value of lane ^ X, X = 1, 2, 4 or 8
template <int X>
__device__ __forceinline__ unsigned lane_xor(unsigned v) {
    if constexpr (X == 1) return __builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
    else if constexpr (X == 2) return __builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
    else if constexpr (X == 4)  // lane ^ 7, then ^ 3
        return __builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF,
                                           true);
    else return __builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);
}

__device__ __forceinline__ void order(unsigned &a, unsigned &b) {
    const unsigned lo = a < b ? a : b, hi = a < b ? b : a;
    a = lo;
    b = hi;
}

// compare with lane ^ X: the lane without bit X keeps the smaller
template <int X, int E>
__device__ __forceinline__ void cross(unsigned (&v)[E], int lane) {
    if constexpr (X >= 16) {
        // rows of two registers swapped so that both partners are in one lane, and back
#pragma unroll
        for (int r = 0; r < E; r += 2) {
            const auto s = X == 16 ? __builtin_amdgcn_permlane16_swap(v[r], v[r + 1], false, false)
                                   : __builtin_amdgcn_permlane32_swap(v[r], v[r + 1], false, false);
            unsigned a = s[0], b = s[1];
            order(a, b);
            const auto q = X == 16 ? __builtin_amdgcn_permlane16_swap(a, b, false, false)
                                   : __builtin_amdgcn_permlane32_swap(a, b, false, false);
            v[r] = q[0];
            v[r + 1] = q[1];
        }
    } else {
        const unsigned lim = lane & X ? ~0u : 0u;
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const unsigned y = lane_xor<X>(v[r]);
            const unsigned lo = v[r] < y ? v[r] : y, hi = v[r] < y ? y : v[r];
            const unsigned m = hi < lim ? hi : lim;  // the middle one of (v, y, lim)
            v[r] = lo > m ? lo : m;
        }
    }
}

// the lane's registers (a bitonic sequence) into ascending order
template <int E>
__device__ __forceinline__ void merge_lane(unsigned (&v)[E]) {
#pragma unroll
    for (int d = E / 2; d > 0; d >>= 1)
#pragma unroll
        for (int r = 0; r < E; ++r)
            if (!(r & d)) order(v[r], v[r + d]);
}

// 64 E keys, E per lane, sorted: lane l gets the E l-th .. of them
template <int E>
__device__ __forceinline__ void sort_wave(unsigned (&v)[E], int lane) {
    // A lane whose keys descend (bit k of the lane, runs of 2^k lanes) holds them
    // complemented, so that every comparison puts the smaller first.
    unsigned flip = (unsigned)-(lane & 1);
#pragma unroll
    for (int r = 0; r < E; ++r) v[r] ^= flip;
    // in the lane: odd-even merge sort (19 comparisons)
#pragma unroll
    for (int p = 1; p < E; p <<= 1)
#pragma unroll
        for (int k = p; k >= 1; k >>= 1)
#pragma unroll
            for (int j = k % p; j + k < E; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (j + i + k < E && (i + j) / (2 * p) == (i + j + k) / (2 * p)) order(v[i + j], v[i + j + k]);
    // runs of 2^(k-1) lanes into runs of 2^k: a loop, not straight-line code, which
    // a launch of a few waves per CU would spend its time fetching
#pragma unroll 1
    for (int k = 1; k <= 6; ++k) {
        const unsigned next = k < 6 ? (unsigned)-(int)((lane >> k) & 1) : 0u;
#pragma unroll
        for (int r = 0; r < E; ++r) v[r] ^= flip ^ next;
        flip = next;
        if (k >= 6) cross<32>(v, lane);
        if (k >= 5) cross<16>(v, lane);
        if (k >= 4) cross<8>(v, lane);
        if (k >= 3) cross<4>(v, lane);
        if (k >= 2) cross<2>(v, lane);
        cross<1>(v, lane);
        merge_lane(v);
    }
}

// slot of sorted entry i of n in the search tree (children of slot k: 2 k, 2 k + 1)
template <int N>
__device__ __forceinline__ int tree_slot(int i) {
    return i == N - 1 ? 0 : (N + i + 1) >> (__builtin_ctz(i + 1) + 1);
}

// One workgroup of W wavefronts: segment blockIdx.y, a tile of 64 E positions = its outputs
// and their median halo of h on either side.  What bounds it is VALU issue, then LDS,
// so the work of a position is shared as far as it goes:
//   the powers (non-negative, so ordered like their bits) are sorted in registers, by
//   the first wavefront;
//   each position's rank is found in a search tree of the sorted keys (levels
//   contiguous: 64 lanes' reads fall on different banks), equal keys taking
//   successive ranks in any order;
//   a lane then slides over consecutive outputs with the set of its window's
//   ranks as bits (64 E per lane, interleaved so that every lane has its own
//   bank): an output removes a rank, adds a rank, and moves the median to the
//   next member up or down, or not at all.
// The W wavefronts share the ranks, the first windows and the outputs; the first one slides.
// 10800 rows of 8000 outputs, window 101, in the first calls after the device idled: 0.90 ms
// (3.07 ms for a workgroup sort in LDS with a count of every sorted block per output);
// tiles of 1024 positions took 1.53: half the waves fit a CU's LDS, and only windows of
// 257 gain what they lose.  With the clocks up 0.73 ms, 95 % of VALU issue.
// The entry is the (h + 1)-th smallest power of the window, exactly.
template <bool SPEC, int E, int W>
__global__ __launch_bounds__(64 * W) void normalise_kernel(const void *__restrict__ rows, int64_t pitch, int64_t k_lo,
                                                           int n_bins, int h, float *__restrict__ out) {
    constexpr int N = 64 * E, kWords = N / 32, kMine = E > W ? E / W : 1;
    __shared__ __attribute__((aligned(16))) unsigned set[kWords * 64];
    __shared__ unsigned tree[N];
    // a rank r as its bit's place: (r / 32) << 8, the word's byte offset among the 64
    // lanes' words, and r % 32 (ordered like the ranks)
    __shared__ unsigned short rank[N], med[N];
    const int lane = threadIdx.x & 63, wv = W > 1 ? threadIdx.x >> 6 : 0;
    const int o0 = blockIdx.x * (N - 2 * h);
    const int n_out = min(N - 2 * h, n_bins - o0);
    const int n_pos = n_out + 2 * h;  // positions that an output reads; the others sort last
    auto power = [&](int p) {
        if constexpr (SPEC)
            return hann_power((const float2 *)rows + (int64_t)blockIdx.y * pitch, k_lo + o0 - h + p, pitch - 1);
        else
            return ((const float *)rows)[(int64_t)blockIdx.y * pitch + o0 + p];
    };
    auto load = [&](int p) { return p < n_pos ? __float_as_uint(power(p)) : ~0u; };
    const bool ranks = kMine * wv < E;  // a wavefront beyond E has none to find
    unsigned key[kMine];
#pragma unroll
    for (int i = 0; i < kMine; ++i) key[i] = ranks ? load(64 * (kMine * wv + i) + lane) : ~0u;
    if (wv == 0) {
        unsigned v[E];
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] = i < kMine ? key[i] : load(64 * i + lane);
        sort_wave(v, lane);
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const int i = lane * E + r;
            tree[r + 1 < E ? (N + i + 1) >> (__builtin_ctz(r + 1) + 1) : tree_slot<N>(i)] = v[r];
        }
    }
    unsigned *const equal = set;  // ranks given out among equal keys
#pragma unroll
    for (int i = wv; i < E; i += W) equal[64 * i + lane] = 0u;
    __syncthreads();
    if (ranks) {
        unsigned at[kMine];
#pragma unroll
        for (int i = 0; i < kMine; ++i) at[i] = 1u;
#pragma unroll 1
        for (int s = 1; s < N; s <<= 1)
#pragma unroll
            for (int i = 0; i < kMine; ++i) at[i] = 2 * at[i] + (tree[at[i]] < key[i] ? 1u : 0u);
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            unsigned r = at[i] - N;
            r += atomicAdd(&equal[r], 1u);
            rank[64 * (kMine * wv + i) + lane] = (unsigned short)((r >> 5 << 8) | (r & 31));
        }
    }
    __syncthreads();
#pragma unroll
    for (int w = wv; w < kWords; w += W) set[w * 64 + lane] = 0u;
    __syncthreads();
    // the lane's outputs first .. first + mine - 1
    const int run = slide_length(n_out);
    const SlideRun own = slide_run(lane, n_out, h);
    const int first = own.first, mine = own.mine;
    char *const bits = reinterpret_cast<char *>(set + lane);
    auto word = [&](int m) -> unsigned & { return *reinterpret_cast<unsigned *>(bits + (m & 0xFF00)); };
    auto toggle = [&](int r) { atomicXor(&word(r), 1u << (r & 31)); };
#pragma unroll 16
    for (int i = wv; i <= 2 * h; i += W) toggle(rank[first + i]);
    if (W > 1) __syncthreads();
    if (wv == 0) {
        int m;  // the median: h members of the set lie below
        {
            int below = 0, at = 0, sum = 0;
#pragma unroll 4
            for (int w = 0; w < kWords; ++w) {
                sum += __popc(set[w * 64 + lane]);
                if (sum <= h) {
                    below = sum;
                    at = w + 1;
                }
            }
            unsigned y = set[at * 64 + lane];
            int k = h - below;
            m = at << 8;
#pragma unroll
            for (int s = 16; s > 0; s >>= 1) {
                const int c = __popc(y & ((1u << s) - 1u));
                if (k >= c) {
                    k -= c;
                    m += s;
                    y >>= s;
                }
            }
        }
        // straight-line, with masks for the lanes that stay: the compiler turns branches
        // here into loops that lanes leave one by one
        const unsigned short *const leave = rank + first, *const enter = rank + own.enter;
        int a = leave[0], b = enter[0];
        for (int s = 0;; ++s) {
            med[first + min(s, mine - 1)] = (unsigned short)m;
            if (s + 1 == run) break;
            const unsigned on = s + 1 < mine ? 1u : 0u;
            atomicXor(&word(a), on << (a & 31));
            atomicXor(&word(b), on << (b & 31));
            // members below m: h, less a's, plus b's
            const int more = (b < m) - (a < m), p = m & 31;
            unsigned x = word(m);
            const bool stay = on == 0u || (more == 0 && a != m);
            const int next = slide_next(s, mine);
            a = leave[next];
            b = enter[next];
            x &= stay ? 1u << p : more > 0 ? (1u << p) - 1u : ~1u << p;
            int w = m & 0xFF00;
            while (x == 0u) {
                w += more > 0 ? -256 : 256;
                x = word(w);
            }
            m = w + (more > 0 ? 31 - __clz((int)x) : __ffs((int)x) - 1);
        }
    }
    __syncthreads();
#pragma unroll 2
    for (int o = threadIdx.x; o < n_out; o += 64 * W) {
        const int m = med[o];
        const float f = __uint_as_float(tree[tree_slot<N>((m >> 8 << 5) | (m & 31))]);
        // rho = P ln2 / median; a window whose median is 0 carries no noise-floor estimate: 0
        const double r = f > 0.0f ? (double)power(o + h) * 0.69314718055994530942 / (double)f : 0.0;
        out[(int64_t)blockIdx.y * n_bins + o0 + o] = (float)r;
    }
}

void sft_release(ltgw_ctx *c) {
    for (auto &pl : c->sft_plans) (void)hipfftDestroy((hipfftHandle)pl.plan);
    c->sft_plans.clear();
    for (auto &t : c->sft_tabs) release(t.tab);
    c->sft_tabs.clear();
    release(c->sft_spec);
    release(c->sft_spec2);
}

}  // namespace ltgw

namespace {

const char *fft_error(hipfftResult r) {
    switch (r) {
        case HIPFFT_ALLOC_FAILED: return "allocation failed";
        case HIPFFT_INVALID_VALUE: return "invalid value";
        case HIPFFT_INVALID_SIZE: return "invalid size";
        case HIPFFT_EXEC_FAILED: return "execution failed";
        case HIPFFT_SETUP_FAILED: return "setup failed";
        default: return "error";
    }
}

}  // namespace

using namespace ltgw;

namespace {

template <bool SPEC, int E, int W>
hipError_t launch_normalise_e(const void *rows, int64_t pitch, int64_t k_lo, int n_bins, int h, int n_seg, float *out,
                              hipStream_t st) {
    const int span = 64 * E - 2 * h;
    const unsigned tiles = (unsigned)((n_bins - 1) / span + 1);
    hipLaunchKernelGGL((normalise_kernel<SPEC, E, W>), dim3(tiles, (unsigned)n_seg), dim3(64 * W), 0, st, rows, pitch,
                       k_lo, n_bins, h, out);
    return hipGetLastError();
}

// rows: powers of the outputs and their halo (float), or raw spectra (float2).  Few tiles
// are a chain of waits, so they are short and their work is shared; many are issue and
// LDS, so the halo counts.  Whole calls, in us, on 256 CUs, with 64 E positions by W
// wavefronts:
//   up to 16 tiles of 128 a CU, where the halo leaves half of one, or one tile a row
//     (64 segments of 700 bins, window 1: 16.2 by <2, 1>, 18.9 by <4, 1>, 27.0 by <8, 1>;
//     4000 of 60, 52.4, 55.1 and 61.2); then 256 (1024 of 7000, window 51: 85.5; <2, 1>
//     139.7, <8, 1> 87.7; window 65: 93.1 and 83.6);
//   up to 6 tiles of 256 a CU, four wavefronts (256 of 700, window 101: 21.6; <4, 1> 23.4,
//     <8, 4> 23.9, <8, 1> 26.4; with 16 a CU 51.0, 48.3, 40.6 and 37.4);
//   up to 3 tiles of 512 a CU, eight (one of 60, window 257: 14.3; <8, 4> 15.5, <8, 1>
//     17.9; 256 of 700, 24.2, 24.4 and 28.0; with 7 a CU 30.1, 26.6 and 31.3);
//   up to 8, four (1000 of 700, window 257: 49.8; <8, 1> 54.2; with 10
//     a CU and window 101 84.6 and 81.9).
template <bool SPEC>
hipError_t launch_normalise(const void *rows, int64_t pitch, int64_t k_lo, int n_bins, int h, int n_seg, int cu_count,
                            float *out, hipStream_t st) {
    auto tiles = [&](int positions) { return ((int64_t)(n_bins - 1) / (positions - 2 * h) + 1) * n_seg; };
    if (2 * h <= 64 && (n_bins <= 128 - 2 * h || tiles(128) <= 16 * cu_count))
        return launch_normalise_e<SPEC, 2, 1>(rows, pitch, k_lo, n_bins, h, n_seg, out, st);
    if (2 * h <= 50) return launch_normalise_e<SPEC, 4, 1>(rows, pitch, k_lo, n_bins, h, n_seg, out, st);
    if (2 * h <= 192 && tiles(256) <= 6 * cu_count)
        return launch_normalise_e<SPEC, 4, 4>(rows, pitch, k_lo, n_bins, h, n_seg, out, st);
    if (tiles(512) <= 3 * cu_count) return launch_normalise_e<SPEC, 8, 8>(rows, pitch, k_lo, n_bins, h, n_seg, out, st);
    if (tiles(512) <= 8 * cu_count) return launch_normalise_e<SPEC, 8, 4>(rows, pitch, k_lo, n_bins, h, n_seg, out, st);
    return launch_normalise_e<SPEC, 8, 1>(rows, pitch, k_lo, n_bins, h, n_seg, out, st);
}

// segments with an on-chip transform: powers of a chunk of segments (about 512 MB), then their ratios
int chip_normalise(ltgw_ctx *c, const float *strain, int n_seg, int n_fft, int64_t k_lo, int n_bins, int h, float *out) {
    int rc;
    const float2 *tab = nullptr;
    for (auto &t : c->sft_tabs)
        if (t.n_fft == n_fft) tab = (const float2 *)t.tab.p;
    if (!tab) {
        DevBuf b;
        if ((rc = ensure(c, b, chip_fft_table_bytes(n_fft), "transform tables")) != LTGW_OK) return rc;
        c->sft_tabs.push_back({n_fft, b});
        tab = (const float2 *)b.p;
        const hipError_t e = launch_chip_fft_tables(n_fft, (float2 *)b.p, c->stream);
        if (e != hipSuccess) {
            release(c->sft_tabs.back().tab);
            c->sft_tabs.pop_back();
            return hip_fail(c, e, "transform tables");
        }
    }
    const int row = n_bins + 2 * h;
    const int batch = (int)std::max<int64_t>(1, std::min<int64_t>(n_seg, ((int64_t)512 << 20) / (4 * (int64_t)row)));
    if ((rc = ensure(c, c->sft_spec, (size_t)batch * row * 4, "powers")) != LTGW_OK) return rc;
    for (int j0 = 0; j0 < n_seg; j0 += batch) {
        const int nb = std::min(batch, n_seg - j0);
        HIP_TRY(c, launch_chip_fft(n_fft, strain + (int64_t)j0 * n_fft, nb, k_lo - h, row, tab, (float *)c->sft_spec.p,
                                   c->stream),
                "transform launch");
        HIP_TRY(c, launch_normalise<false>(c->sft_spec.p, row, k_lo, n_bins, h, nb, c->cu_count,
                                          out + (int64_t)j0 * n_bins, c->stream),
                "normalise launch");
    }
    return LTGW_OK;
}

}  // namespace

// A chunk of strain rows (n_fft reals each) into the transform buffer's rows
// of n_fft + 2 reals: 8-byte moves (n_fft is even, so every row of both is
// 8-byte aligned), a grid-stride loop over each row.
__global__ __launch_bounds__(256) void pad_rows_kernel(const float2 *__restrict__ src, int64_t src_pitch,
                                                       float2 *__restrict__ dst, int64_t dst_pitch, int64_t pairs) {
    const float2 *s = src + (int64_t)blockIdx.y * src_pitch;
    float2 *d = dst + (int64_t)blockIdx.y * dst_pitch;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < pairs; i += (int64_t)gridDim.x * 256) d[i] = s[i];
}

extern "C" {

int32_t ltgw_sft_normalise(ltgw_ctx *c, const float *strain, int32_t n_seg, int32_t n_fft, int64_t k_lo,
                           int32_t n_bins, int32_t window, float *out) {
    if (!c) return LTGW_E_INVALID_ARG;
    Enter en(c);
    if (!strain || !out) return fail(c, LTGW_E_INVALID_ARG, "strain or out is NULL");
    if (!is_device_ptr(strain) || !is_device_ptr(out))
        return fail(c, LTGW_E_INVALID_ARG, "strain and out must be device memory");
    if (n_seg < 1 || n_seg > 65535) return fail(c, LTGW_E_INVALID_ARG, "n_seg must be in 1 .. 65535");
    if (n_fft < 2 || (n_fft & 1) || n_fft > (1 << 24))
        return fail(c, LTGW_E_INVALID_ARG, "n_fft must be even and in 2 .. 2^24");
    if (window < 1 || !(window & 1) || window > kSftMaxWindow)
        return fail(c, LTGW_E_INVALID_ARG, "window must be odd and in 1 .. %d", kSftMaxWindow);
    const int h = window / 2;
    if (n_bins < 1 || k_lo < h || k_lo + n_bins - 1 + h > n_fft / 2)
        return fail(c, LTGW_E_INVALID_ARG, "band [k_lo - window/2, k_lo + n_bins - 1 + window/2] must lie in 0 .. n_fft/2");
    if (chip_fft_has(n_fft)) return chip_normalise(c, strain, n_seg, n_fft, k_lo, n_bins, h, out);
    int rc;
    // chunks of segments: spectra within about 512 MB
    const int64_t per_seg = (int64_t)(n_fft / 2 + 1) * 8;
    int batch = (int)std::max<int64_t>(1, std::min<int64_t>(n_seg, ((int64_t)512 << 20) / per_seg));
    if ((rc = ensure(c, c->sft_spec, (size_t)batch * (n_fft / 2 + 1) * 8, "spectra")) != LTGW_OK) return rc;
    // More than one chunk: alternate two spectra buffers, and normalise on the
    // side stream, so that a chunk's normalisation (VALU issue) overlaps the
    // next chunk's copy and transform (HBM-bound).  The copy into a buffer
    // waits for the normalisation that last read it; the context's stream
    // waits for the last normalisations before the call's work ends.
    const bool two = n_seg > batch;
    if (two && (rc = ensure(c, c->sft_spec2, (size_t)batch * (n_fft / 2 + 1) * 8, "spectra")) != LTGW_OK)
        return rc;
    int k = 0;
    for (int j0 = 0; j0 < n_seg; j0 += batch, ++k) {
        const int nb = std::min(batch, n_seg - j0);
        const int b = k & 1;
        void *const spec = b ? c->sft_spec2.p : c->sft_spec.p;
        // a plan per (n_fft, batch size), kept for later calls
        hipfftHandle plan = nullptr;
        for (auto &pl : c->sft_plans)
            if (pl.n_fft == n_fft && pl.batch == nb) plan = (hipfftHandle)pl.plan;
        if (!plan) {
            // in place: rows of n_fft + 2 reals in, n_fft / 2 + 1 complex out
            int n = n_fft, in_len = n_fft + 2, out_len = n_fft / 2 + 1;
            const hipfftResult r = hipfftPlanMany(&plan, 1, &n, &in_len, 1, n_fft + 2, &out_len, 1, n_fft / 2 + 1,
                                                  HIPFFT_R2C, nb);
            if (r != HIPFFT_SUCCESS) return fail(c, LTGW_E_DEVICE, "FFT plan: %s", fft_error(r));
            c->sft_plans.push_back({n_fft, nb, (void *)plan});
        }
        // the chunk's segments are copied into the spectra buffer (rows padded
        // to n_fft + 2 reals) and transformed there in place: the library's
        // transform may use its input as scratch, and the caller's strain is
        // only read
        if (two && k >= 2) HIP_TRY(c, hipStreamWaitEvent(c->stream, c->ev_sft[2 + b], 0), "spectra reuse");
        {
            const int64_t pairs = n_fft / 2;
            const unsigned gx = (unsigned)std::min<int64_t>((pairs + 255) / 256, 16);
            hipLaunchKernelGGL(pad_rows_kernel, dim3(gx, (unsigned)nb), dim3(256), 0, c->stream,
                               (const float2 *)(strain + (int64_t)j0 * n_fft), pairs, (float2 *)spec,
                               (int64_t)(n_fft / 2 + 1), pairs);
            HIP_TRY(c, hipGetLastError(), "strain copy launch");
        }
        hipfftResult r = hipfftSetStream(plan, c->stream);
        if (r == HIPFFT_SUCCESS) r = hipfftExecR2C(plan, (hipfftReal *)spec, (hipfftComplex *)spec);
        if (r != HIPFFT_SUCCESS) return fail(c, LTGW_E_DEVICE, "FFT: %s", fft_error(r));
        hipStream_t ns = c->stream;
        if (two) {
            HIP_TRY(c, hipEventRecord(c->ev_sft[b], c->stream), "event record");
            HIP_TRY(c, hipStreamWaitEvent(c->side, c->ev_sft[b], 0), "normalise order");
            ns = c->side;
        }
        HIP_TRY(c, launch_normalise<true>(spec, n_fft / 2 + 1, k_lo, n_bins, h, nb, c->cu_count,
                                         out + (int64_t)j0 * n_bins, ns),
                "normalise launch");
        if (two) HIP_TRY(c, hipEventRecord(c->ev_sft[2 + b], c->side), "event record");
    }
    if (two)
        for (int b = 0; b < 2 && b < k; ++b)
            HIP_TRY(c, hipStreamWaitEvent(c->stream, c->ev_sft[2 + b], 0), "normalise join");
    return LTGW_OK;
}

}  // extern "C"
