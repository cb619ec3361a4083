// HIP kernels (gfx950) for the template-bank detection statistic.
//
// Data layout in HBM
//   store   per detector, [n_seg][pitch] elements of 4/2/1 bytes (FP32, BF16,
//           OCP E4M3).  Element 0 and element n_bins+1 of every row are 0
//           guards; element b+1 holds column b.  The sign bit of each element
//           is the number-count bit (rho > rho_th, decided on the FP32 input):
//           normalised power is non-negative, so the bit is free and one
//           gather serves both statistics (Sec. 2: power and number count).
//   H       per detector, [n_sky][n_brake][n_tau][n_seg] FP64,
//           H = RN(RN(g*D)*T_sft), the bin-scaled ratio f^/f0 of Eqs. 1-2.
//   results per template: s (FP64), c, N (int32), W1, W2 (FP64).
//
// Evaluation kernel: one lane per template, 256 consecutive f0 per block,
// one (sky, n, tau) group per block row.  Per segment a lane does
//   x = f0*H (FP64)  v = x + (1.5 - k_lo)  i = (unsigned)trunc(v)
// and gathers element i of the segment's row with a structured buffer load
// (idxen; stride = element size; the row as the scalar byte offset).  The
// resource holds n_bins + 2 records, so the hardware range check returns 0
// for every index past the upper guard, including negative ones (large as
// unsigned).  Neighbouring f0 lanes read neighbouring
// columns, so a wavefront's 64 gathers fall in a few cache lines.  The
// per-segment H, weight and row address are wavefront-uniform (SGPRs).
// trunc(v) - 1 equals floor(RN(x + 0.5)) - k_lo whenever the latter is in
// band, for k_lo >= 2 and x < 2^30 (both checked by the host): x + 1.5 - k_lo
// is exact in FP64 whenever its magnitude is at most x, and every other case
// lands on the lower guard or out of range.
#include <algorithm>
#include <cmath>

#include "ltgw_gather.h"
#include "ltgw_internal.h"
#include "ddpow.h"

#pragma clang fp contract(off)

namespace ltgw {

// ---------------------------------------------------------------------------
// Ingest: FP32 power -> store with guards and the count bit.
__device__ inline unsigned bf16_rne_bits(float x) {  // finite x >= 0
    unsigned u = __float_as_uint(x);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
__device__ inline unsigned e4m3_rne_sat_bits(float a) {  // finite a >= 0
    if (!(a < 448.0f)) return 0x7eu;
    unsigned u = __float_as_uint(a);
    int ex = (int)(u >> 23) - 127;
    if (ex < -6) return (unsigned)__builtin_rintf(a * 512.0f);  // m * 2^-9, m <= 8
    unsigned keep = (u >> 20) & 7u, rem = u & 0xfffffu;
    if (rem > 0x80000u || (rem == 0x80000u && (keep & 1u))) keep += 1u;
    return ((unsigned)(ex + 7) << 3) + keep;
}

__device__ inline float block_max_256(float v, float *sh) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    float m = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
    __syncthreads();
    return m;
}

template <int STORE>
__global__ __launch_bounds__(256) void ingest_kernel(const float *__restrict__ in, int n_bins,
                                                     int64_t pitch, void *__restrict__ out,
                                                     float *__restrict__ scale,
                                                     const float *__restrict__ w, int w_rows,
                                                     float *__restrict__ wq, float th,
                                                     unsigned long long *bad) {
    __shared__ float sh[4];
    const int64_t j = blockIdx.x;
    const float *row = in + j * (int64_t)n_bins;
    float sc = 1.0f;
    if (STORE == LTGW_STORE_FP8) {
        float m = 0.0f;
        for (int b = threadIdx.x; b < n_bins; b += 256) {
            float x = row[b];
            if (x >= 0.0f && x <= 3.402823466e38f) m = fmaxf(m, x);
        }
        m = block_max_256(m, sh);
        sc = (m == 0.0f) ? 1.0f : m / 448.0f;
    }
    unsigned nbad = 0;
    for (int64_t b = threadIdx.x; b < pitch; b += 256) {
        unsigned code = 0;
        if (b >= 1 && b <= n_bins) {
            float x = row[b - 1];
            if (!(x >= 0.0f && x <= 3.402823466e38f)) {
                ++nbad;
                x = 0.0f;
            }
            x = __builtin_fabsf(x);  // -0 -> +0
            unsigned bit = x > th ? 1u : 0u;
            if (STORE == LTGW_STORE_F32) code = __float_as_uint(x) | (bit << 31);
            if (STORE == LTGW_STORE_BF16) code = bf16_rne_bits(x) | (bit << 15);
            if (STORE == LTGW_STORE_FP8) code = e4m3_rne_sat_bits(x / sc) | (bit << 7);
        }
        if (STORE == LTGW_STORE_F32) ((unsigned *)out)[j * pitch + b] = code;
        if (STORE == LTGW_STORE_BF16) ((unsigned short *)out)[j * pitch + b] = (unsigned short)code;
        if (STORE == LTGW_STORE_FP8) ((unsigned char *)out)[j * pitch + b] = (unsigned char)code;
    }
    if (nbad) atomicAdd(bad, (unsigned long long)nbad);
    if (threadIdx.x == 0) {
        scale[j] = sc;
        wq[j] = w[j % w_rows] * sc;
    }
}

hipError_t launch_ingest(int store, const float *power, int32_t n_seg, int32_t n_bins,
                         int64_t pitch, void *out, float *scale, const float *w, int32_t w_rows, float *wq,
                         float rho_th, unsigned long long *bad, hipStream_t st) {
    dim3 grid(n_seg), block(256);
    if (store == LTGW_STORE_F32)
        hipLaunchKernelGGL(ingest_kernel<LTGW_STORE_F32>, grid, block, 0, st, power, n_bins, pitch,
                           out, scale, w, w_rows, wq, rho_th, bad);
    else if (store == LTGW_STORE_BF16)
        hipLaunchKernelGGL(ingest_kernel<LTGW_STORE_BF16>, grid, block, 0, st, power, n_bins, pitch,
                           out, scale, w, w_rows, wq, rho_th, bad);
    else
        hipLaunchKernelGGL(ingest_kernel<LTGW_STORE_FP8>, grid, block, 0, st, power, n_bins, pitch,
                           out, scale, w, w_rows, wq, rho_th, bad);
    return hipGetLastError();
}

// Stack ingest with the proposer's coarse store in the same pass: workgroup
// (j2, r) reads the S fine rows S j2 .. S j2 + S - 1 of realisation r once and
//  - writes them to the fine store: the codes, count bits and FP8 scales of
//    ingest_kernel, bit for bit;
//  - writes coarse pixel m of coarse row j2 (column m + 1; columns 0 and
//    nb2 + 1 .. pitch2 - 1 are 0 guards): the FP32 sum, segment by segment in
//    order, of the pair sums P[2m] + P[2m+1], rounded to bfloat16, in the
//    upper half of a 32-bit word whose low byte counts the 2 S pixels of the
//    block above rho_th (the fine count bits; at most 16).
// With crs NULL only the fine store is written (S rows per workgroup).
template <int STORE>
__global__ __launch_bounds__(256) void stack_ingest_kernel(const float *__restrict__ in, int n_seg, int n_bins,
                                                           int S, int64_t pitch, void *__restrict__ out,
                                                           float *__restrict__ scale, const float *__restrict__ w,
                                                           float *__restrict__ wq, float th, int64_t pitch2,
                                                           unsigned *__restrict__ crs, unsigned long long *bad) {
    __shared__ float sh[4];
    __shared__ float ssc[8];
    const int j2 = blockIdx.x, r = blockIdx.y;
    const int ns2 = n_seg / S, nb2 = n_bins / 2;
    const int64_t row0 = (int64_t)r * n_seg + (int64_t)S * j2;  // first fine row of the block
    for (int k = 0; k < S; ++k) {
        float sc = 1.0f;
        if (STORE == LTGW_STORE_FP8) {
            const float *row = in + (row0 + k) * n_bins;
            float m = 0.0f;
            for (int b = threadIdx.x; b < n_bins; b += 256) {
                const float x = row[b];
                if (x >= 0.0f && x <= 3.402823466e38f) m = fmaxf(m, x);
            }
            m = block_max_256(m, sh);
            sc = (m == 0.0f) ? 1.0f : m / 448.0f;
        }
        if (threadIdx.x == 0) {
            ssc[k] = sc;
            scale[row0 + k] = sc;
            wq[row0 + k] = w[S * j2 + k] * sc;  // one realisation's weights serve all
        }
    }
    __syncthreads();
    unsigned nbad = 0;
    unsigned *co = crs ? crs + ((int64_t)r * ns2 + j2) * pitch2 : nullptr;
    for (int m = threadIdx.x; m < nb2; m += 256) {
        float acc = 0.0f;
        unsigned cnt = 0;
        for (int k = 0; k < S; ++k) {
            const float *src = in + (row0 + k) * n_bins + 2 * m;
            float x[2] = {src[0], src[1]};
            unsigned code[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (!(x[e] >= 0.0f && x[e] <= 3.402823466e38f)) {
                    ++nbad;
                    x[e] = 0.0f;
                }
                x[e] = __builtin_fabsf(x[e]);  // -0 -> +0
                const unsigned bit = x[e] > th ? 1u : 0u;
                cnt += bit;
                if (STORE == LTGW_STORE_F32) code[e] = __float_as_uint(x[e]) | (bit << 31);
                if (STORE == LTGW_STORE_BF16) code[e] = bf16_rne_bits(x[e]) | (bit << 15);
                if (STORE == LTGW_STORE_FP8) code[e] = e4m3_rne_sat_bits(x[e] / ssc[k]) | (bit << 7);
            }
            const float pair = x[0] + x[1];
            acc = k == 0 ? pair : acc + pair;
            const int64_t o = (row0 + k) * pitch + 2 * m + 1;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (STORE == LTGW_STORE_F32) ((unsigned *)out)[o + e] = code[e];
                if (STORE == LTGW_STORE_BF16) ((unsigned short *)out)[o + e] = (unsigned short)code[e];
                if (STORE == LTGW_STORE_FP8) ((unsigned char *)out)[o + e] = (unsigned char)code[e];
            }
        }
        if (co) co[m + 1] = (bf16_rne_bits(acc) << 16) | cnt;
    }
    // the guards: fine columns 0 and n_bins + 1 .. pitch - 1 of the S rows,
    // coarse columns 0 and nb2 + 1 .. pitch2 - 1
    const int64_t gf = pitch - n_bins;  // guard columns per fine row
    for (int64_t e = threadIdx.x; e < (int64_t)S * gf; e += 256) {
        const int64_t k = e / gf, q = e % gf;
        const int64_t o = (row0 + k) * pitch + (q == 0 ? 0 : n_bins + q);
        if (STORE == LTGW_STORE_F32) ((unsigned *)out)[o] = 0u;
        if (STORE == LTGW_STORE_BF16) ((unsigned short *)out)[o] = 0;
        if (STORE == LTGW_STORE_FP8) ((unsigned char *)out)[o] = 0;
    }
    if (co)
        for (int64_t q = threadIdx.x; q < pitch2 - nb2; q += 256) co[q == 0 ? 0 : nb2 + q] = 0u;
    if (nbad) atomicAdd(bad, (unsigned long long)nbad);
}

hipError_t launch_stack_ingest(int store, const float *power, int R, int32_t n_seg, int32_t n_bins, int S,
                               int64_t pitch, void *out, float *scale, const float *w, float *wq, float rho_th,
                               int64_t pitch2, unsigned *crs, unsigned long long *bad, hipStream_t st) {
    if (R < 1 || R > 65535 || S < 1 || S > 8 || n_seg % S || (n_bins & 1) || pitch < n_bins + 2 ||
        (crs && pitch2 < n_bins / 2 + 2))
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)(n_seg / S), (unsigned)R), block(256);
#define LTGW_STACK_INGEST(ST)                                                                                   \
    hipLaunchKernelGGL(stack_ingest_kernel<ST>, grid, block, 0, st, power, n_seg, n_bins, S, pitch, out, scale, \
                       w, wq, rho_th, pitch2, crs, bad)
    if (store == LTGW_STORE_F32)
        LTGW_STACK_INGEST(LTGW_STORE_F32);
    else if (store == LTGW_STORE_BF16)
        LTGW_STACK_INGEST(LTGW_STORE_BF16);
    else
        LTGW_STACK_INGEST(LTGW_STORE_FP8);
#undef LTGW_STACK_INGEST
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Eq. 1: g[(i_n*n_tau + i_tau)][j] = RN(u^e), 0 where t_j < T0.
__global__ __launch_bounds__(256) void spin_factor_kernel(const double *__restrict__ t_seg,
                                                          int n_seg, double t0,
                                                          const double *__restrict__ tau,
                                                          int n_tau,
                                                          const double *__restrict__ brake,
                                                          double *__restrict__ g,
                                                          unsigned long long *pow_counts) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    const int grp = blockIdx.y;
    if (j >= n_seg) return;
    const double t = t_seg[j];
    double out = 0.0;
    if (!(t < t0)) {
        const double ta = tau[grp % n_tau];
        const double n = brake[grp / n_tau];
        const double d = t - t0;
        const double q = d / ta;
        const double u = 1.0 + q;
        const double e = 1.0 / (1.0 - n);
        int und = 0;
        int slow = 0;
        out = pow_cr(u, e, &und, &slow);
        if (und) atomicAdd(pow_counts, 1ull);
        if (slow) atomicAdd(pow_counts + 1, 1ull);
    }
    g[(int64_t)grp * n_seg + j] = out;
}

hipError_t launch_spin_factor(const double *t_seg, int32_t n_seg, double t0, const double *tau,
                              int32_t n_tau, const double *brake, int32_t n_brake, double *g,
                              unsigned long long *pow_counts, hipStream_t st) {
    dim3 grid((n_seg + 255) / 256, n_tau * n_brake), block(256);
    hipLaunchKernelGGL(spin_factor_kernel, grid, block, 0, st, t_seg, n_seg, t0, tau, n_tau, brake,
                       g, pow_counts);
    return hipGetLastError();
}

// Eq. 2 and the bin scale: H[(sky*n_tn + tn)][j] = RN(RN(g*D)*T_sft),
// D = 1 + ((vx nx + vy ny) + vz nz)/c.
__global__ __launch_bounds__(256) void track_factor_kernel(const double *__restrict__ g,
                                                           int n_tn,
                                                           const double *__restrict__ v,
                                                           int n_seg,
                                                           const double *__restrict__ sky,
                                                           double t_sft, double *__restrict__ H) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    const int row = blockIdx.y;  // sky * n_tn + tn
    if (j >= n_seg) return;
    const int s = row / n_tn, tn = row % n_tn;
    const double a = v[3 * j + 0] * sky[3 * s + 0];
    const double b = v[3 * j + 1] * sky[3 * s + 1];
    const double z = v[3 * j + 2] * sky[3 * s + 2];
    const double vn = (a + b) + z;
    const double r = vn / kC;
    const double D = 1.0 + r;
    const double h = g[(int64_t)tn * n_seg + j] * D;
    H[(int64_t)row * n_seg + j] = h * t_sft;
}

hipError_t launch_track_factor(const double *g, int32_t n_tn, const double *v, int32_t n_seg,
                               const double *sky, int32_t n_sky, double t_sft, double *H,
                               hipStream_t st) {
    dim3 grid((n_seg + 255) / 256, n_sky * n_tn), block(256);
    hipLaunchKernelGGL(track_factor_kernel, grid, block, 0, st, g, n_tn, v, n_seg, sky, t_sft, H);
    return hipGetLastError();
}

// A launch covers the segments [j_lo, j_hi) (a slab; multiples of the chunk
// except a final j_hi = n_seg): a slab after the first resumes from the sums
// the previous slab stored (the same operations in the same order as one
// pass), and only the last slab writes the caller's outputs.
template <int STORE, bool MOMENTS, int TPL, int U>
__global__ __launch_bounds__(256) void eval_kernel(const EvalArgs a, int first, int total, int j_lo, int j_hi,
                                                   int last) {
    const int n_tiles = (a.n_f0 + 256 * TPL - 1) / (256 * TPL);
    int tile, grp;
    xcd_tile_group(blockIdx.x, gridDim.x, n_tiles, tile, grp, first, total);
    int i[TPL];
    double f0[TPL];
    for (int t = 0; t < TPL; ++t) {
        i[t] = tile * 256 * TPL + t * 256 + threadIdx.x;
        f0[t] = a.f0_min + (double)i[t] * a.f0_step;
    }
    Acc<TPL> acc;
    acc.zero();
    if (j_lo > 0)
        for (int t = 0; t < TPL; ++t) {
            if (i[t] >= a.n_f0) continue;
            const int64_t q = (int64_t)grp * a.n_f0 + i[t];
            acc.s[t] = a.s[q];
            acc.cnt[t] = a.c[q];
            if (MOMENTS) {
                acc.nin[t] = a.n[q];
                acc.w1[t] = a.w1[q];
                acc.w2[t] = a.w2[q];
            }
        }
    for (int d = 0; d < a.n_det; ++d) {
        DetView D = a.det[d];
        if (D.w_sky_stride) {  // antenna-pattern weights: the row of this group's sky point
            const int64_t off = (int64_t)(grp / a.n_tn) * D.w_sky_stride;
            D.wq += off;
            D.w += off;
        }
        int jb, je;
        const int runs = D.win ? 256 * TPL / D.win_run : 1;
        seg_window(D, grp, tile * runs, (tile + 1) * runs, jb, je);
        jb = jb > j_lo ? jb : j_lo;
        je = je < j_hi ? je : j_hi;
        if (jb < je)
            accumulate_det<STORE, MOMENTS, TPL, U>(D, HTable{D.H + (int64_t)grp * D.n_seg}, f0, acc, jb, je);
    }
    store_results<MOMENTS, TPL>(acc, i, grp, a.n_f0, a.s, a.c, a.n, a.w1, a.w2, last ? a.out_s : nullptr,
                                last ? a.out_c : nullptr, last ? a.out_n : nullptr,
                                last ? a.in_band_total : nullptr);
}

// The same with the segments shared: 64 templates per workgroup, its wavefronts a chunk
// of segments each, and the first wavefront adds the chunk sums in their order, so the
// bits are the same.  A lane of eval_kernel walks all its segments alone: with few
// templates most of the chip is idle, with more the longest walks are what a launch
// waits for (12 x 400 templates over 1024 segments: 58 us there, 10 here).
template <int STORE, bool MOMENTS, int kSplitWaves>
__global__ __launch_bounds__(64 * kSplitWaves) void eval_split_kernel(const EvalArgs a) {
    __shared__ SharedSums<MOMENTS, 1, kSplitWaves> part;
    __shared__ int count[MOMENTS ? 2 : 1][1][kSplitWaves][64];
    const int n_tiles = (a.n_f0 + 63) / 64;
    const int tile = (int)blockIdx.x % n_tiles, grp = (int)blockIdx.x / n_tiles;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i[1] = {tile * 64 + ((int)threadIdx.x & 63)};
    const double f0[1] = {a.f0_min + (double)i[0] * a.f0_step};
    Acc<1> acc;
    acc.zero();
    int b = 0;
    for (int d = 0; d < a.n_det; ++d) {
        DetView D = a.det[d];
        if (D.w_sky_stride) {  // antenna-pattern weights: the row of this group's sky point
            const int64_t off = (int64_t)(grp / a.n_tn) * D.w_sky_stride;
            D.wq += off;
            D.w += off;
        }
        int jb, je;
        const int run = D.win ? tile * 64 / D.win_run : 0;
        seg_window(D, grp, run, run + 1, jb, je);
        accumulate_shared<STORE, MOMENTS, 1, 16, kSplitWaves>(D, HTable{D.H + (int64_t)grp * D.n_seg}, f0, acc, jb, je, wv,
                                                              part, b);
    }
    add_counts<MOMENTS, 1, kSplitWaves>(acc, wv, count);
    if (wv != 0) return;
    store_results<MOMENTS, 1>(acc, i, grp, a.n_f0, a.s, a.c, a.n, a.w1, a.w2, a.out_s, a.out_c, a.out_n,
                              a.in_band_total);
}

// How many wavefronts share 64 templates, 0 for eval_kernel.  By n = (f0 / 64) x groups:
// with n below two workgroups a CU 16 (n = 300 of 10000 FP32 segments: 70 us, 101 with
// 8, 171 with 4, 529 in eval_kernel), then 8 (n = 756 of 3000 BF16: 50 us, 67 with 16,
// 61 with 4, 160), then 4 (n = 5304 of 2 x 2699 BF16: 307 us; 603).  The workgroups in
// flight walk different rows, so the more columns they cover the less their caches
// serve: eval_kernel, whose order keeps an XCD on few columns, is level at n x bytes of
// the lattice's columns in a row of 40 - 60 MB (8000 FP32 columns: 258 us against 264
// at n = 1500, 818 against 499 at 4500; 4000 BF16: 305 against 355 at 5040, 593 against
// 549 at 9072; with moments in the loop 4000 FP8: 471 against 488 at 9072).  One or two chunks of segments
// are nothing to share: eval_kernel's larger workgroups start sooner (500 f0 x 600 groups
// of 32 segments: 14.5 us against 17.7, 1990 x 140 of 64 11.6 against 15.6).
int eval_split_waves(int store, int n_seg, int n_f0, int64_t n_groups, int cu_count) {
    if (n_seg <= 2 * kChunk) return 0;
    const int64_t n = (int64_t)((n_f0 + 63) / 64) * n_groups;
    const int bytes = store == LTGW_STORE_F32 ? 4 : store == LTGW_STORE_BF16 ? 2 : 1;
    if (n * n_f0 * bytes > 40000000) return 0;
    return n <= 2 * cu_count ? 16 : n <= 5 * cu_count ? 8 : 4;
}

template <int STORE, bool MOMENTS>
static hipError_t launch_eval_split_m(int waves, const EvalArgs &a, hipStream_t st) {
    const int64_t n = (int64_t)((a.n_f0 + 63) / 64) * a.n_groups;
    if (n < 1 || n > 0x7fffffff) return hipErrorInvalidValue;
    if (waves == 16)
        hipLaunchKernelGGL((eval_split_kernel<STORE, MOMENTS, 16>), dim3((unsigned)n), dim3(64 * 16), 0, st, a);
    else if (waves == 8)
        hipLaunchKernelGGL((eval_split_kernel<STORE, MOMENTS, 8>), dim3((unsigned)n), dim3(64 * 8), 0, st, a);
    else
        hipLaunchKernelGGL((eval_split_kernel<STORE, MOMENTS, 4>), dim3((unsigned)n), dim3(64 * 4), 0, st, a);
    return hipGetLastError();
}

template <int STORE>
static hipError_t launch_eval_split_s(bool moments, int waves, const EvalArgs &a, hipStream_t st) {
    return moments ? launch_eval_split_m<STORE, true>(waves, a, st) : launch_eval_split_m<STORE, false>(waves, a, st);
}

hipError_t launch_eval_split(int store, bool moments, int waves, const EvalArgs &a, hipStream_t st) {
    if (store == LTGW_STORE_F32) return launch_eval_split_s<LTGW_STORE_F32>(moments, waves, a, st);
    if (store == LTGW_STORE_BF16) return launch_eval_split_s<LTGW_STORE_BF16>(moments, waves, a, st);
    return launch_eval_split_s<LTGW_STORE_FP8>(moments, waves, a, st);
}

// Tile shapes: (templates per lane, segments per gather batch).
constexpr int kVariantTpl[kNumShapes] = {1, 1, 2, 2};

int variant_templates_per_block(int variant) { return 256 * kVariantTpl[variant & 3]; }

// Segments per slab (variant & 8); a multiple of the chunk.
constexpr int kSlab = 1024;

template <int STORE, bool MOMENTS, int TPL, int U>
static hipError_t launch_eval_v(const EvalArgs &a, bool generations, bool slabs, int cu_count, hipStream_t st,
                                int *launches) {
    *launches = 0;
    const int64_t blocks = (int64_t)((a.n_f0 + 256 * TPL - 1) / (256 * TPL)) * a.n_groups;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    int64_t step = blocks;
    if (generations) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, eval_kernel<STORE, MOMENTS, TPL, U>, 256, 0) !=
                hipSuccess || per_cu < 1) {
            (void)hipGetLastError();
            per_cu = 1;
        }
        step = (int64_t)cu_count * per_cu;
    }
    // slabs only for one detector (one segment axis)
    const int n_seg = a.det[0].n_seg;
    const int slab = (slabs && a.n_det == 1) ? kSlab : 0x7fffffff;
    for (int j_lo = 0; j_lo == 0 || j_lo < n_seg; j_lo += slab) {
        const int j_hi = (a.n_det > 1 || slab == 0x7fffffff || j_lo + slab >= n_seg) ? 0x7fffffff : j_lo + slab;
        const int last = j_hi == 0x7fffffff ? 1 : 0;
        for (int64_t first = 0; first < blocks; first += step) {
            const int64_t n = blocks - first < step ? blocks - first : step;
            hipLaunchKernelGGL((eval_kernel<STORE, MOMENTS, TPL, U>), dim3((unsigned)n), dim3(256), 0, st, a,
                               (int)first, (int)blocks, j_lo, j_hi, last);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            ++*launches;
        }
        if (last) break;
    }
    return hipSuccess;
}

template <int STORE, bool MOMENTS>
static hipError_t launch_eval_m(int variant, const EvalArgs &a, int cu_count, hipStream_t st, int *launches) {
    const bool gen = (variant & 4) != 0, slabs = (variant & 8) != 0;
    switch (variant & 3) {
        case 0: return launch_eval_v<STORE, MOMENTS, 1, 8>(a, gen, slabs, cu_count, st, launches);
        case 1: return launch_eval_v<STORE, MOMENTS, 1, 16>(a, gen, slabs, cu_count, st, launches);
        case 2: return launch_eval_v<STORE, MOMENTS, 2, 8>(a, gen, slabs, cu_count, st, launches);
        default: return launch_eval_v<STORE, MOMENTS, 2, 16>(a, gen, slabs, cu_count, st, launches);
    }
}

template <int STORE>
static hipError_t launch_eval_s(bool moments, int variant, const EvalArgs &a, int cu_count, hipStream_t st,
                                int *launches) {
    return moments ? launch_eval_m<STORE, true>(variant, a, cu_count, st, launches)
                   : launch_eval_m<STORE, false>(variant, a, cu_count, st, launches);
}

hipError_t launch_eval(int store, bool moments, int variant, const EvalArgs &a, int cu_count, hipStream_t st,
                       int *launches) {
    if (variant < 0 || variant >= kNumVariants) return hipErrorInvalidValue;
    if (store == LTGW_STORE_F32) return launch_eval_s<LTGW_STORE_F32>(moments, variant, a, cu_count, st, launches);
    if (store == LTGW_STORE_BF16) return launch_eval_s<LTGW_STORE_BF16>(moments, variant, a, cu_count, st, launches);
    return launch_eval_s<LTGW_STORE_FP8>(moments, variant, a, cu_count, st, launches);
}

// ---------------------------------------------------------------------------
// Many searches in one persistent launch.  Tiles (search, group, 64 x TPL
// consecutive f0) are listed largest search first; every resident workgroup
// takes the next tile from an atomic counter until the list is exhausted (the
// loop ends for every workgroup once the counter passes the tile count), its
// wavefronts sharing the tile's segments.  The workgroup that finishes a search's
// last tile stamps the search's completion time.
// 41000 tiles of 64 f0, 2.2e9 in-band evaluations: 1.07 ms with a tile per workgroup, 1.29
// with one per wavefront (the last ones walked alone).  Counting the tiles through a
// generic pointer, 64 flat atomics each on one address, had made it 17.0 ms.
template <int STORE, bool MOMENTS, int TPL, int U>
__global__ __launch_bounds__(256) void batch_kernel(const BatchArgs a) {
    constexpr int kWaves = 4;
    __shared__ SharedSums<MOMENTS, TPL, kWaves> part;
    __shared__ int count[MOMENTS ? 2 : 1][TPL][kWaves][64];
    __shared__ int ticket;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (threadIdx.x == 0 && a.t_start) atomicMin(a.t_start, (unsigned long long)wall_clock64());
    int b = 0;
    // No lane-divergent branch stands around the hand-out or at the loop's end: the
    // first wavefront's lanes all issue the atomic (lane 0 adds 1, the others 0; through
    // a global pointer that is one atomic) and all write the ticket.  With a lane-0-only
    // branch there the compiler once split the loop, parking lane 0 while the other
    // lanes went round with a stale ticket.
    for (;;) {
        __syncthreads();  // the last tile's reads of LDS
        if (wv == 0) {
            const unsigned t = atomicAdd(a.counter, lane == 0 ? 1u : 0u);
            ticket = __builtin_amdgcn_readfirstlane((int)t);
        }
        __syncthreads();
        const int tt = __builtin_amdgcn_readfirstlane(ticket);
        if (tt >= a.n_tiles) break;
        // descriptors are read into scalar registers (uniform loop bounds, buffer
        // resources and table pointers)
        const BatchTile T = uniform(a.tiles[tt]);
        const BatchSearch *Sp = a.searches + T.search;
        const int n_det = uniform(Sp->n_det), n_f0 = uniform(Sp->n_f0), n_tn = uniform(Sp->n_tn);
        const double f0_min = uniform(Sp->f0_min), f0_step = uniform(Sp->f0_step);
        int i[TPL];
        double f0[TPL];
        for (int t = 0; t < TPL; ++t) {
            i[t] = T.tile * 64 * TPL + t * 64 + lane;
            f0[t] = f0_min + (double)i[t] * f0_step;
        }
        const int tn = T.grp % n_tn, sky = T.grp / n_tn;
        Acc<TPL> acc;
        acc.zero();
        for (int d = 0; d < n_det; ++d) {
            const DetView D = uniform(Sp->det[d]);
            const HFromGD hs{D.g + (int64_t)tn * D.n_seg, D.D + (int64_t)sky * D.n_seg, D.t_sft};
            int jb, je;
            const int runs = D.win ? 64 * TPL / D.win_run : 1;  // the batch's windows are per 64 f0
            seg_window(D, T.grp, T.tile * runs, (T.tile + 1) * runs, jb, je);
            accumulate_shared<STORE, MOMENTS, TPL, U, kWaves>(D, hs, f0, acc, jb, je, wv, part, b);
        }
        add_counts<MOMENTS, TPL, kWaves>(acc, wv, count);
        if (wv != 0) continue;
        store_results<MOMENTS, TPL>(acc, i, T.grp, n_f0, uniform(Sp->s), uniform(Sp->c), uniform(Sp->n),
                                    uniform(Sp->w1), uniform(Sp->w2), nullptr, nullptr, nullptr,
                                    a.in_band_total);
        // the tile's stores have left the wave before it counts as done; later kernels
        // of the stream read them, so no cache is written back here
        __builtin_amdgcn_s_waitcnt(0);
        typedef __attribute__((address_space(1))) unsigned GlobalCount;
        GlobalCount *const tiles_done = (GlobalCount *)(uintptr_t)uniform(Sp->tiles_done);
        unsigned long long *const t_done = uniform(Sp->t_done);
        const unsigned done = (unsigned)__builtin_amdgcn_readfirstlane(
                                  (int)__hip_atomic_fetch_add(tiles_done, lane == 0 ? 1u : 0u, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT)) + 1u;
        if (done == (unsigned)uniform(Sp->n_tiles) && t_done) *t_done = wall_clock64();  // same value, every lane
    }
}

template <int STORE, bool MOMENTS, int TPL, int U>
static hipError_t launch_batch_v(const BatchArgs &a, int grid, hipStream_t st) {
    hipLaunchKernelGGL((batch_kernel<STORE, MOMENTS, TPL, U>), dim3(grid), dim3(256), 0, st, a);
    return hipGetLastError();
}

template <int STORE, bool MOMENTS>
static hipError_t launch_batch_m(int variant, const BatchArgs &a, int grid, hipStream_t st) {
    switch (variant & 3) {
        case 0: return launch_batch_v<STORE, MOMENTS, 1, 8>(a, grid, st);
        case 1: return launch_batch_v<STORE, MOMENTS, 1, 16>(a, grid, st);
        case 2: return launch_batch_v<STORE, MOMENTS, 2, 8>(a, grid, st);
        default: return launch_batch_v<STORE, MOMENTS, 2, 16>(a, grid, st);
    }
}

hipError_t launch_batch(int store, bool moments, int variant, const BatchArgs &a, int grid,
                        hipStream_t st) {
    if (store == LTGW_STORE_F32)
        return moments ? launch_batch_m<LTGW_STORE_F32, true>(variant, a, grid, st)
                       : launch_batch_m<LTGW_STORE_F32, false>(variant, a, grid, st);
    if (store == LTGW_STORE_BF16)
        return moments ? launch_batch_m<LTGW_STORE_BF16, true>(variant, a, grid, st)
                       : launch_batch_m<LTGW_STORE_BF16, false>(variant, a, grid, st);
    return moments ? launch_batch_m<LTGW_STORE_FP8, true>(variant, a, grid, st)
                   : launch_batch_m<LTGW_STORE_FP8, false>(variant, a, grid, st);
}

int batch_blocks_per_cu(int store, bool moments, int variant) {
    int n = 0;
    hipError_t e = hipSuccess;
#define LTGW_OCC(S, M, T, U)                                                                    \
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, batch_kernel<S, M, T, U>, 256, 0)
#define LTGW_OCC_V(S, M)                            \
    switch (variant & 3) {                          \
        case 0: LTGW_OCC(S, M, 1, 8); break;        \
        case 1: LTGW_OCC(S, M, 1, 16); break;       \
        case 2: LTGW_OCC(S, M, 2, 8); break;        \
        default: LTGW_OCC(S, M, 2, 16); break;      \
    }
    if (store == LTGW_STORE_F32) {
        if (moments) { LTGW_OCC_V(LTGW_STORE_F32, true) } else { LTGW_OCC_V(LTGW_STORE_F32, false) }
    } else if (store == LTGW_STORE_BF16) {
        if (moments) { LTGW_OCC_V(LTGW_STORE_BF16, true) } else { LTGW_OCC_V(LTGW_STORE_BF16, false) }
    } else {
        if (moments) { LTGW_OCC_V(LTGW_STORE_FP8, true) } else { LTGW_OCC_V(LTGW_STORE_FP8, false) }
    }
#undef LTGW_OCC_V
#undef LTGW_OCC
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return n < 1 ? 1 : n;
}

// Eq. 2 table for batched searches: D[sky][j] = 1 + ((vx nx + vy ny) + vz nz)/c.
__global__ __launch_bounds__(256) void doppler_kernel(const double *__restrict__ v, int n_seg,
                                                      const double *__restrict__ sky,
                                                      double *__restrict__ D) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    const int s = blockIdx.y;
    if (j >= n_seg) return;
    const double a = v[3 * j + 0] * sky[3 * s + 0];
    const double b = v[3 * j + 1] * sky[3 * s + 1];
    const double z = v[3 * j + 2] * sky[3 * s + 2];
    const double vn = (a + b) + z;
    const double r = vn / kC;
    D[(int64_t)s * n_seg + j] = 1.0 + r;
}

// In-band segment windows.  For a segment, the column index trunc(f0 h +
// 1.5 - k_lo) is non-decreasing in f0, so a run of consecutive f0 has a lane
// in band exactly when its last f0 reaches column 1 and its first f0 is at
// most column n_bins.  A window may be wider than that (segments out of band add
// exact zeros), so the columns are formed in FP32 and compared with a margin of
// 2^-20 of the terms, four times what their rounding can come to.  f0 goes in times
// the power of two that brings the largest below 1 and the track factors divided by it,
// so that neither leaves FP32's range, whatever the unit of time: columns stay below
// 2^30, and a term that underflows is far below the first column.
// One wavefront per (group, kWinRuns consecutive runs of f0): each lane takes
// segments lane, lane + 64, ... and tests every run of the wavefront against
// its track factor, so the group's row of track factors is read once per
// kWinRuns runs; each run's first and last in-band segment are then reduced
// across the wavefront.  80 groups of 5400 segments, 4000 f0: 29 us (46 with FP64
// columns and one track factor in flight).
constexpr int kWinRuns = 8;
__global__ __launch_bounds__(256) void window_kernel(const DetView D, int n_groups, int n_tn, double f0_min,
                                                     double f0_step, int n_f0, double h_scale,
                                                     int2 *__restrict__ win) {
    const int lane = threadIdx.x & 63;
    const int per_group = (D.win_blocks + 4 * kWinRuns - 1) / (4 * kWinRuns);
    const int grp = blockIdx.x / per_group;
    const int blk0 = ((blockIdx.x % per_group) * 4 + (threadIdx.x >> 6)) * kWinRuns;
    if (blk0 >= D.win_blocks) return;
    float fa[kWinRuns], fb[kWinRuns];
    int lo[kWinRuns], hi[kWinRuns];
#pragma unroll
    for (int r = 0; r < kWinRuns; ++r) {
        const int ia = (blk0 + r) * D.win_run;
        const int ib = min(ia + D.win_run - 1, n_f0 - 1);
        fa[r] = (float)(f0_min + (double)ia * f0_step);
        fb[r] = (float)(f0_min + (double)ib * f0_step);
        lo[r] = D.n_seg;
        hi[r] = -1;
    }
    const float c = (float)D.cshift, top = (float)(f0_min + (double)(n_f0 - 1) * f0_step);
    const float past = (float)D.n_bins + 1.0f;
    const int tn = grp % n_tn, sky = grp / n_tn;
    for (int j0 = lane; j0 < D.n_seg; j0 += 4 * 64) {
        float h[4];  // four track factors in flight
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = min(j0 + 64 * k, D.n_seg - 1);
            if (D.H) {
                h[k] = (float)(D.H[(int64_t)grp * D.n_seg + j] * h_scale);
            } else {
                const double hg = D.g[(int64_t)tn * D.n_seg + j] * D.D[(int64_t)sky * D.n_seg + j];
                h[k] = (float)(hg * D.t_sft * h_scale);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = min(j0 + 64 * k, D.n_seg - 1);  // the last segment again changes nothing
            const float margin = 0x1p-20f * (top * h[k] + __builtin_fabsf(c) + past);
            const float from = 1.0f - margin, to = past + margin;
#pragma unroll
            for (int r = 0; r < kWinRuns; ++r)
                if (__builtin_fmaf(fb[r], h[k], c) >= from && __builtin_fmaf(fa[r], h[k], c) <= to) {
                    lo[r] = min(lo[r], j);
                    hi[r] = max(hi[r], j);
                }
        }
    }
#pragma unroll
    for (int r = 0; r < kWinRuns; ++r) {
        int l = lo[r], u = hi[r];
        for (int o = 32; o > 0; o >>= 1) {
            l = min(l, __shfl_xor(l, o, 64));
            u = max(u, __shfl_xor(u, o, 64));
        }
        if (lane == 0 && blk0 + r < D.win_blocks) win[(int64_t)grp * D.win_blocks + blk0 + r] = make_int2(l, u);
    }
}

hipError_t launch_windows(const DetView &D, int n_groups, int n_tn, double f0_min, double f0_step, int n_f0,
                          int2 *win, hipStream_t st) {
    const int64_t blocks = (int64_t)((D.win_blocks + 4 * kWinRuns - 1) / (4 * kWinRuns)) * n_groups;
    if (n_groups < 1 || D.win_blocks < 1 || blocks > 0x7fffffff) return hipErrorInvalidValue;
    int ex = 0;  // (both powers of two are doubles of full precision)
    (void)std::frexp(f0_min + (double)(n_f0 - 1) * f0_step, &ex);
    ex = std::min(std::max(ex, -1000), 1000);
    const double down = std::ldexp(1.0, -ex);
    hipLaunchKernelGGL(window_kernel, dim3((unsigned)blocks), dim3(256), 0, st, D, n_groups, n_tn, f0_min * down,
                       f0_step * down, n_f0, std::ldexp(1.0, ex), win);
    return hipGetLastError();
}

hipError_t launch_doppler(const double *v, int32_t n_seg, const double *sky, int32_t n_sky,
                          double *D, hipStream_t st) {
    hipLaunchKernelGGL(doppler_kernel, dim3((n_seg + 255) / 256, n_sky), dim3(256), 0, st, v, n_seg,
                       sky, D);
    return hipGetLastError();
}

__global__ void fill_u32_kernel(unsigned *p, int n, unsigned v) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) p[i] = v;
}
__global__ void fill_u64_kernel(unsigned long long *p, int n, unsigned long long v) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) p[i] = v;
}

hipError_t launch_fill_u32(unsigned *p, int n, unsigned v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024), dim3(256),
                       0, st, p, n, v);
    return hipGetLastError();
}
__global__ void f64_to_f32_kernel(const double *in, float *out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        out[i] = (float)in[i];
}

hipError_t launch_f64_to_f32(const double *in, float *out, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(f64_to_f32_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, st,
                       in, out, n);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, int n, unsigned long long v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u64_kernel, dim3((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024), dim3(256),
                       0, st, p, n, v);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// In-band moments (N, W1, W2) without touching the spectrogram.  For a fixed
// (group, segment) the column index trunc(f0_i*H + 1.5 - k_lo) is a
// non-decreasing function of i (every step is monotone), so the in-band
// templates are the contiguous range [lo, hi) with lo the first i whose
// index reaches 1 and hi the first whose index passes n_bins.  Both are
// found by binary search with exactly the statistic kernel's arithmetic.
__device__ inline int col_index(double f0_min, double f0_step, int i, double H, double cshift) {
    const double f0 = f0_min + (double)i * f0_step;
    const double x = f0 * H;
    const double vv = x + cshift;
    return __double2int_rz(vv);
}

// first i in [0, n] with col_index(i) >= target (n if none), looked for at `near`:
// column target starts at f0 H = target - cshift, so i = ((target - cshift) / H -
// f0_min) / f0_step but for rounding, and the columns on either side confirm it.
// Where they don't (steps near the rounding of f0, no step at all), a binary search.
__device__ inline int first_at_least(double f0_min, double f0_step, int n, double H,
                                     double cshift, int target, double near) {
    // (a NaN clamps to 0)
    const int i = (int)__builtin_fmin(__builtin_fmax(__builtin_ceil(near), 0.0), (double)n);
    const bool before = col_index(f0_min, f0_step, i - 1, H, cshift) >= target && i > 0;
    const bool here = col_index(f0_min, f0_step, i, H, cshift) >= target || i == n;
    if (here && !before) return i;
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (col_index(f0_min, f0_step, mid, H, cshift) >= target)
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// T threads per (group, part of the f0), R groups a workgroup: the range ends of every
// segment added into differences in LDS (integers: any order gives the same sums), and the
// prefix sums of those.  Ends below the part count at its start, which most segments
// share, so those are summed in registers; ends beyond it count nowhere.
// Differences in device memory with binary searches, 32 segments a lane, took 54 us for
// 12 groups of 1024 segments (this: 6), 95 and a 9 us scan for 456 groups of two times
// 4465 (28), and beside the statistic, with four sums a template, 1.22 ms and a scan
// of 0.47 ms for 288 groups of 10800 (113 us alone).
template <int NA, int T>
constexpr int kMomPart = 8 * T / NA;  // f0 of a part: with 512 threads 32 KB of differences

template <int NA, int T, int R>
__global__ __launch_bounds__(T *R) void moments_kernel(const EvalArgs a, int e0) {
    __shared__ unsigned long long diffs[R][NA][kMomPart<NA, T>];
    __shared__ unsigned long long parts[R][NA][T / 64];
    __shared__ unsigned long long in_band;
    const int sub = R > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / T) : 0, tid = R > 1 ? threadIdx.x % T : threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    auto &diff = diffs[sub];
    auto &part = parts[sub];
    const bool mine = (int)blockIdx.y * R + sub < a.n_groups;  // the others take its last group along
    const int row = mine ? blockIdx.y * R + sub : a.n_groups - 1;
    const int i0 = blockIdx.x * kMomPart<NA, T>, i1 = min(i0 + kMomPart<NA, T>, a.n_f0);
    for (int k = tid; k < i1 - i0; k += T)
#pragma unroll
        for (int q = 0; q < NA; ++q) diff[q][k] = 0ull;
    if (threadIdx.x == 0) in_band = 0ull;
    __syncthreads();
    const int tn = row % a.n_tn, sky = row / a.n_tn;
    const double per_step = 1.0 / a.f0_step;
    unsigned long long inb = 0, at0[NA];
#pragma unroll
    for (int q = 0; q < NA; ++q) at0[q] = 0ull;
    for (int d = 0; d < a.n_det; ++d) {
        const DetView &D = a.det[d];
        for (int j4 = tid; j4 < D.n_seg; j4 += 4 * T) {
            double h4[4];  // four track factors in flight
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = min(j4 + k * T, D.n_seg - 1);
                if (D.H) {
                    h4[k] = D.H[(int64_t)row * D.n_seg + j];
                } else {
                    const double h = D.g[(int64_t)tn * D.n_seg + j] * D.D[(int64_t)sky * D.n_seg + j];
                    h4[k] = h * D.t_sft;
                }
            }
#pragma unroll 1
            for (int k = 0; k < 4; ++k) {
                const int j = j4 + k * T;
                if (j >= D.n_seg) break;
                const double H = k == 0 ? h4[0] : k == 1 ? h4[1] : k == 2 ? h4[2] : h4[3];
                // 1 / H to about 2^-50: where to look, no more
                double inv = __builtin_amdgcn_rcp(H);
                inv = __builtin_fma(__builtin_fma(-H, inv, 1.0), inv, inv);
                inv = __builtin_fma(__builtin_fma(-H, inv, 1.0), inv, inv);
                const int lo = max(i0, first_at_least(a.f0_min, a.f0_step, a.n_f0, H, D.cshift, 1,
                                                      ((1.0 - D.cshift) * inv - a.f0_min) * per_step));
                const int hi = min(i1, first_at_least(a.f0_min, a.f0_step, a.n_f0, H, D.cshift, D.n_bins + 1,
                                                      (((double)D.n_bins + 1.0 - D.cshift) * inv - a.f0_min) * per_step));
                if (lo >= hi) continue;
                inb += (unsigned long long)(hi - lo);
                unsigned long long val[NA];
                val[0] = 1ull;
#pragma unroll
                for (int q = 1; q < NA; ++q) val[q] = (unsigned long long)D.wfix[3 * j + q - 1];
#pragma unroll
                for (int q = 0; q < NA; ++q) {
                    if (lo == i0)
                        at0[q] += val[q];
                    else
                        atomicAdd(&diff[q][lo - i0], val[q]);
                    if (hi < i1) atomicAdd(&diff[q][hi - i0], 0ull - val[q]);
                }
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        inb += __shfl_xor(inb, o, 64);
#pragma unroll
        for (int q = 0; q < NA; ++q) at0[q] += __shfl_xor(at0[q], o, 64);
    }
    if (lane == 0) {
        if (mine && inb) atomicAdd(&in_band, inb);
#pragma unroll
        for (int q = 0; q < NA; ++q) atomicAdd(&diff[q][0], at0[q]);
    }
    __syncthreads();
    // one addition per workgroup to the search's total: they queue at its address, 12 ns
    // each (25,000 from the wavefronts of 3150 workgroups were all of a launch's 311 us; with
    // a workgroup for each of 60000 groups of 64 segments, 1 f0, the evaluation took 907 us,
    // with eight groups a workgroup 424; a loop over groups took 438, but twice the
    // registers beside a batch, 1166 ms against 985 for 64 searches)
    if (threadIdx.x == 0 && in_band && a.in_band_total) atomicAdd(a.in_band_total, in_band);
    // each thread's run of consecutive f0: its sum, the sums before it, its prefix sums
    const int per = (i1 - i0 + T - 1) / T;
    const int k0 = tid * per, k1 = min(k0 + per, i1 - i0);
    int64_t run[NA];
#pragma unroll
    for (int q = 0; q < NA; ++q) {
        int64_t v = 0;
        for (int k = k0; k < k1; ++k) v += (int64_t)diff[q][k];
        int64_t u = v;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t w = __shfl_up(u, o, 64);
            if (lane >= o) u += w;
        }
        if (lane == 63) part[q][wv] = (unsigned long long)u;
        run[q] = u - v;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NA; ++q)
        for (int k = 0; k < wv; ++k) run[q] += (int64_t)part[q][k];
    const double wu = (double)a.w_uniform;
    const int64_t t0 = (int64_t)row * a.n_f0 + i0;
    auto put = [&](int k, const int64_t (&r)[NA]) {
        if (!mine) return;
        const int nin = (int)r[0];
        double w1, w2;
        if constexpr (NA > 1) {
            w1 = ldexp((double)r[1], e0);
            w2 = ldexp((double)r[2] * 4294967296.0 + (double)r[3], 2 * e0);
        } else {
            w1 = (double)nin * wu;
            w2 = (double)nin * (wu * wu);
        }
        a.n[t0 + k] = nin;
        a.w1[t0 + k] = w1;
        a.w2[t0 + k] = w2;
        if (a.out_n) a.out_n[t0 + k] = nin;
    };
    if (per == 1) {
        if (k0 < k1) {
#pragma unroll
            for (int q = 0; q < NA; ++q) run[q] += (int64_t)diff[q][k0];
            put(k0, run);
        }
        return;
    }
    // runs: the sums back to their places, from where neighbouring lanes write neighbouring
    // templates (a thread's run of 8 written by itself, 64 bytes from the next one's, took a
    // search of 17 million templates of 3 segments 594 us, so 317)
    for (int k = k0; k < k1; ++k)
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            run[q] += (int64_t)diff[q][k];
            diff[q][k] = (unsigned long long)run[q];
        }
    __syncthreads();
    for (int k = tid; k < i1 - i0; k += T) {
        int64_t r[NA];
#pragma unroll
        for (int q = 0; q < NA; ++q) r[q] = (int64_t)diff[q][k];
        put(k, r);
    }
}

template <int T, int R>
static hipError_t launch_moments_t(const EvalArgs &a, int weights, int e0, hipStream_t st) {
    const int per = weights ? kMomPart<4, T> : kMomPart<1, T>;
    const dim3 grid((unsigned)((a.n_f0 - 1) / per + 1), (unsigned)((a.n_groups - 1) / R + 1));
    if (weights)
        hipLaunchKernelGGL((moments_kernel<4, T, R>), grid, dim3(T * R), 0, st, a, e0);
    else
        hipLaunchKernelGGL((moments_kernel<1, T, R>), grid, dim3(T * R), 0, st, a, e0);
    return hipGetLastError();
}

// 64 threads a group where the groups fill the chip and one part of them holds the f0:
// with 512 most of them wait for segments (60000 groups of 64 segments, the evaluation: 1 f0
// 424 us, 656 with 512, weighted 453 and 1078), while for fewer groups the segments are
// the work to share (300 groups of 5000 segments: 128 us with 64, 104 with 512), and so are
// parts (weighted, 5000 f0 x 300 groups of 1000 segments: 209 and 177).
hipError_t launch_moments(const EvalArgs &a, int weights, int e0, hipStream_t st) {
    if (a.n_groups >= 2048 && a.n_f0 <= (weights ? kMomPart<4, 64> : kMomPart<1, 64>))
        return launch_moments_t<64, 8>(a, weights, e0, st);
    return launch_moments_t<512, 1>(a, weights, e0, st);
}

// ---------------------------------------------------------------------------
// Eq. 4 critical ratios.
__device__ inline double psi_of(uint32_t stat, int64_t t, const double *s, const int32_t *c,
                                const int32_t *N, const double *w1, const double *w2, double q) {
    const int32_t nn = N[t];
    if (nn == 0) return __builtin_nan("");
    if (stat == LTGW_STAT_POWER) {
        const double num = s[t] - w1[t];
        return num / sqrt(w2[t]);
    }
    const double Nq = (double)nn * q;
    const double num = (double)c[t] - Nq;
    const double var = Nq * (1.0 - q);
    return num / sqrt(var);
}

__global__ __launch_bounds__(256) void psi_kernel(uint32_t stat, int64_t n, const double *s,
                                                  const int32_t *c, const int32_t *N,
                                                  const double *w1, const double *w2, double q,
                                                  double *out) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < n) out[t] = psi_of(stat, t, s, c, N, w1, w2, q);
}

hipError_t launch_psi(uint32_t stat, int64_t n, const double *s, const int32_t *c,
                      const int32_t *N, const double *w1, const double *w2, double q,
                      double *out, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(psi_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, stat, n, s,
                       c, N, w1, w2, q, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Top-k by (psi desc, index asc).  For k > kTopkFast: a block takes 4096 items
// into registers (16 per lane) and extracts its k best by k rounds of a block-wide
// arg-max; levels repeat over the per-block winners until one block remains.
constexpr int kTopkIpt = 16;
constexpr int kTopkChunk = 256 * kTopkIpt;
constexpr int64_t kNoIndex = 0x7fffffffffffffffll;

__device__ inline bool better(double pa, int64_t ia, double pb, int64_t ib) {
    return pa > pb || (pa == pb && ia < ib);
}

template <bool FROM_RESULTS>
__global__ __launch_bounds__(256) void topk_level_kernel(
    int64_t n, int32_t k, uint32_t stat, const double *s, const int32_t *c, const int32_t *N,
    const double *w1, const double *w2, double q, const double *in_psi, const int64_t *in_idx,
    double *out_psi, int64_t *out_idx) {
    __shared__ double sp[4];
    __shared__ int64_t si[4];
    double pv[kTopkIpt];
    int64_t iv[kTopkIpt];
    const int64_t base = (int64_t)blockIdx.x * kTopkChunk;
#pragma unroll
    for (int u = 0; u < kTopkIpt; ++u) {
        const int64_t t = base + (int64_t)u * 256 + threadIdx.x;
        double p = -__builtin_inf();
        int64_t id = kNoIndex;
        if (t < n) {
            if (FROM_RESULTS) {
                p = psi_of(stat, t, s, c, N, w1, w2, q);
                id = t;
            } else {
                p = in_psi[t];
                id = in_idx[t];
            }
            if (!(p == p) || id == kNoIndex) {  // NaN: never ranks
                p = -__builtin_inf();
                id = kNoIndex;
            }
        }
        pv[u] = p;
        iv[u] = id;
    }
    for (int r = 0; r < k; ++r) {
        double bp = -__builtin_inf();
        int64_t bi = kNoIndex;
#pragma unroll
        for (int u = 0; u < kTopkIpt; ++u)
            if (iv[u] != kNoIndex && better(pv[u], iv[u], bp, bi)) {
                bp = pv[u];
                bi = iv[u];
            }
        for (int o = 32; o > 0; o >>= 1) {
            const double op = __shfl_xor(bp, o, 64);
            const int64_t oi = __shfl_xor(bi, o, 64);
            if (oi != kNoIndex && (bi == kNoIndex || better(op, oi, bp, bi))) {
                bp = op;
                bi = oi;
            }
        }
        if ((threadIdx.x & 63) == 0) {
            sp[threadIdx.x >> 6] = bp;
            si[threadIdx.x >> 6] = bi;
        }
        __syncthreads();
        bp = sp[0];
        bi = si[0];
        for (int wv = 1; wv < 4; ++wv)
            if (si[wv] != kNoIndex && (bi == kNoIndex || better(sp[wv], si[wv], bp, bi))) {
                bp = sp[wv];
                bi = si[wv];
            }
        // block-uniform values from LDS, made scalar so the early exit below
        // is a uniform branch (barriers inside the loop)
        bi = ((int64_t)__builtin_amdgcn_readfirstlane((int)(bi >> 32)) << 32) |
             (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)bi);
        __syncthreads();
        if (threadIdx.x == 0) {
            out_psi[(int64_t)blockIdx.x * k + r] = bp;
            out_idx[(int64_t)blockIdx.x * k + r] = bi;
        }
        if (bi == kNoIndex) {
            // no valid item left: pad the rest
            for (int r2 = r + 1 + (int)threadIdx.x; r2 < k; r2 += 256) {
                out_psi[(int64_t)blockIdx.x * k + r2] = -__builtin_inf();
                out_idx[(int64_t)blockIdx.x * k + r2] = kNoIndex;
            }
            break;
        }
#pragma unroll
        for (int u = 0; u < kTopkIpt; ++u)
            if (iv[u] == bi) {
                iv[u] = kNoIndex;
                pv[u] = -__builtin_inf();
            }
    }
}

// The record of ranked template t (kNoIndex: none).
__device__ inline ltgw_candidate topk_record(uint32_t stat, int64_t t, double psi, const double *s, const int32_t *c,
                                             const int32_t *N, const TopkDecode &dec) {
    ltgw_candidate rec;
    if (t == kNoIndex) {
        rec.index = -1;
        rec.f0 = rec.tau = rec.brake = rec.stat = rec.psi = 0.0;
        rec.sky = -1;
        rec.n_valid = 0;
        return rec;
    }
    if (dec.list) {
        const ltgw_template &T = dec.list[t];
        rec.f0 = T.f0;
        rec.tau = T.tau;
        rec.brake = T.brake;
        rec.sky = -1;
    } else {
        const int64_t i_f0 = t % dec.n_f0;
        const int64_t grp = t / dec.n_f0;
        const int64_t i_tau = grp % dec.n_tau;
        const int64_t rr = grp / dec.n_tau;
        rec.f0 = dec.f0_min + (double)i_f0 * dec.f0_step;
        rec.tau = dec.tau[i_tau];
        rec.brake = dec.brake[rr % dec.n_brake];
        rec.sky = (int32_t)(rr / dec.n_brake);
    }
    rec.index = t;
    rec.n_valid = N[t];
    rec.stat = stat == LTGW_STAT_POWER ? s[t] : (double)c[t];
    rec.psi = psi;
    return rec;
}

__global__ void topk_records_kernel(int32_t k, uint32_t stat, const double *s, const int32_t *c,
                                    const int32_t *N, const double *psi, const int64_t *idx,
                                    TopkDecode dec, ltgw_candidate *out, int32_t *n_out) {
    const int r = threadIdx.x;
    if (r == 0) {
        int cntv = 0;
        for (int u = 0; u < k; ++u)
            if (idx[u] != kNoIndex) ++cntv;
        *n_out = cntv;
    }
    if (r < k) out[r] = topk_record(stat, idx[r], psi[r], s, c, N, dec);
}

// For k <= kTopkFast, one launch for the whole ranking (and, with gridDim.y = 2,
// for the second job too): each workgroup ranks its share of the templates, the
// last one to finish ranks the workgroups' winners and writes the records.
// A tile of 4096 items is ranked without k rounds of block-wide reductions: the
// best of each group of 16 lanes is taken first; the k-th best of those 64 bounds
// the k-th best item from below, so only items at or above it (those of at most k
// groups, usually little more than k items) go to a list, whose ranks are counted
// directly.  Later tiles only list items better than the running k-th.
// A workgroup per CU at most, so that for k up to 16 the last one ranks every
// winner as a single tile (512 workgroups of 256 lanes left it five tiles one after
// the other, 47 us at 2.3 million templates).  4800 templates, k = 10: 33 + 17 + 6 us
// in three launches -> 13 us in one; 2.3 million: 45 + 2 x 22 + 6 -> 35 us.
constexpr int kTopkFast = 32;
constexpr int kTopkBlocks = 256;
constexpr int kTopkItems = 4;                         // per lane and tile
constexpr int kTopkTile = 1024 * kTopkItems;
constexpr int kTopkGroup = 16;                        // lanes per group

struct TopkEntry {
    double p;
    int64_t i;
};
__device__ inline bool better(const TopkEntry &a, const TopkEntry &b) { return better(a.p, a.i, b.p, b.i); }

struct TopkShared {
    TopkEntry best[kTopkFast];  // the running winners, best first
    TopkEntry group[64];
    TopkEntry list[kTopkFast * kTopkGroup * kTopkItems + kTopkFast];
    TopkEntry bound;
    int n_best, n_list, n_group, last;
};

// Rank the tile's items (index kNoIndex: none) against the running winners.
__device__ inline void topk_tile(TopkShared &S, int k, const TopkEntry (&it)[kTopkItems]) {
    const int t = threadIdx.x;
    const bool full = S.n_best == k;
    const TopkEntry floor_ = full ? S.best[k - 1] : TopkEntry{-__builtin_inf(), kNoIndex};
    TopkEntry m{-__builtin_inf(), kNoIndex};
#pragma unroll
    for (int u = 0; u < kTopkItems; ++u)
        if (it[u].i != kNoIndex && (!full || better(it[u], floor_)) && (m.i == kNoIndex || better(it[u], m))) m = it[u];
#pragma unroll
    for (int o = 1; o < kTopkGroup; o <<= 1) {
        const TopkEntry x{__shfl_xor(m.p, o, 64), (int64_t)__shfl_xor((long long)m.i, o, 64)};
        if (x.i != kNoIndex && (m.i == kNoIndex || better(x, m))) m = x;
    }
    if (t == 0) S.n_list = S.n_group = 0;
    const int sub = t & (kTopkGroup - 1);
    if (sub == 0) S.group[t / kTopkGroup] = m;
    __syncthreads();
    if (m.i != kNoIndex && sub == 0) atomicAdd(&S.n_group, 1);
    // rank of this group among the 64, a sixteenth of the comparisons per lane
    int rank = 0;
#pragma unroll
    for (int u = 0; u < 64 / kTopkGroup; ++u) {
        const TopkEntry x = S.group[u * kTopkGroup + sub];
        rank += x.i != kNoIndex && better(x, m) ? 1 : 0;
    }
#pragma unroll
    for (int o = 1; o < kTopkGroup; o <<= 1) rank += __shfl_xor(rank, o, 64);
    if (m.i != kNoIndex && rank == k - 1) S.bound = m;  // the same value from the group's lanes
    __syncthreads();
    const int n_group = S.n_group;
    if (n_group == 0) {  // uniform: nothing beats the running winners
        __syncthreads();
        return;
    }
    const bool bounded = n_group >= k;
    const TopkEntry bound = S.bound;
#pragma unroll
    for (int u = 0; u < kTopkItems; ++u)
        if (it[u].i != kNoIndex && (!full || better(it[u], floor_)) && !(bounded && better(bound, it[u])))
            S.list[atomicAdd(&S.n_list, 1)] = it[u];
    if (t < S.n_best) S.list[atomicAdd(&S.n_list, 1)] = S.best[t];
    __syncthreads();
    const int n = S.n_list;
    for (int e0 = 0; e0 < n; e0 += 64) {
        const int e = e0 + t / kTopkGroup;
        const TopkEntry x = S.list[e < n ? e : 0];
        int r = 0;
        for (int u = sub; u < n; u += kTopkGroup) r += better(S.list[u], x) ? 1 : 0;
#pragma unroll
        for (int o = 1; o < kTopkGroup; o <<= 1) r += __shfl_xor(r, o, 64);
        if (e < n && sub == 0 && r < k) S.best[r] = x;
    }
    if (t == 0) S.n_best = n < k ? n : k;
    __syncthreads();
}

__global__ __launch_bounds__(1024) void topk_kernel(const TopkJob j0, const TopkJob j1, int32_t k) {
    __shared__ TopkShared S;
    const TopkJob &J = blockIdx.y ? j1 : j0;
    const int t = threadIdx.x;
    if (t == 0) S.n_best = 0;
    __syncthreads();
    TopkEntry it[kTopkItems];
    for (int64_t base = (int64_t)blockIdx.x * kTopkTile; base < J.n; base += (int64_t)gridDim.x * kTopkTile) {
        // every load of the tile is issued before any ratio is formed (a branch on
        // N per item, as in psi_of, would make them one round trip each)
        const bool power = J.stat == LTGW_STAT_POWER;
        int32_t N[kTopkItems];
        double x[kTopkItems], w1[kTopkItems], w2[kTopkItems];
#pragma unroll
        for (int u = 0; u < kTopkItems; ++u) {
            const int64_t i = base + u * 1024 + t, at = i < J.n ? i : J.n - 1;
            N[u] = J.N[at];
            if (power) {
                x[u] = J.s[at];
                w1[u] = J.w1[at];
                w2[u] = J.w2[at];
            } else {
                x[u] = (double)J.c[at];
                w1[u] = (double)N[u] * J.q;
                w2[u] = w1[u] * (1.0 - J.q);
            }
        }
#pragma unroll
        for (int u = 0; u < kTopkItems; ++u) {
            const int64_t i = base + u * 1024 + t;
            const double p = (x[u] - w1[u]) / sqrt(w2[u]);  // psi_of's operations
            it[u] = TopkEntry{-__builtin_inf(), kNoIndex};
            if (i < J.n && N[u] != 0 && p == p) it[u] = TopkEntry{p, i};  // no segment or NaN: never ranks
        }
        topk_tile(S, k, it);
    }
    if (gridDim.x > 1) {
        TopkEntry *cand = (TopkEntry *)J.cand;
        if (t < k) cand[(int64_t)blockIdx.x * k + t] = t < S.n_best ? S.best[t] : TopkEntry{-__builtin_inf(), kNoIndex};
        // the first wavefront wrote the winners; its first lane publishes them (one
        // release per workgroup: a fence in every wavefront writes its L2 back each time)
        if (t == 0) {
            S.last = __hip_atomic_fetch_add(J.done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1 ? 1 : 0;
            if (S.last) *J.done = 0u;  // for the next launch
            S.n_best = 0;
        }
        __syncthreads();
        if (!S.last) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const int n = (int)gridDim.x * k;
        for (int base = 0; base < n; base += kTopkTile) {
#pragma unroll
            for (int u = 0; u < kTopkItems; ++u) {
                const int i = base + u * 1024 + t;
                it[u] = i < n ? cand[i] : TopkEntry{-__builtin_inf(), kNoIndex};
            }
            topk_tile(S, k, it);
        }
    }
    if (t < k) {
        const TopkEntry x = t < S.n_best ? S.best[t] : TopkEntry{0.0, kNoIndex};
        J.out[t] = topk_record(J.stat, x.i, x.p, J.s, J.c, J.N, J.dec);
    }
    if (t == 0) *J.n_out = S.n_best;
}

int64_t topk_scratch_entries(int64_t n, int32_t k) {
    if (k <= kTopkFast) return std::min<int64_t>((n + kTopkTile - 1) / kTopkTile, kTopkBlocks) * k;
    return 2 * ((n + kTopkChunk - 1) / kTopkChunk * (int64_t)k + k);
}

hipError_t launch_topk(int n_jobs, const TopkJob *jobs, int32_t k, int64_t cand_cap, hipStream_t st) {
    if (n_jobs < 1 || n_jobs > 2 || k < 1) return hipErrorInvalidValue;
    for (int q = 0; q < n_jobs; ++q)
        if (jobs[q].n != jobs[0].n || topk_scratch_entries(jobs[q].n, k) > cand_cap) return hipErrorInvalidValue;
    const int64_t n = jobs[0].n;
    if (k <= kTopkFast) {
        const int64_t tiles = std::max<int64_t>(1, (n + kTopkTile - 1) / kTopkTile);
        const dim3 grid((unsigned)std::min<int64_t>(tiles, kTopkBlocks), (unsigned)n_jobs);
        hipLaunchKernelGGL(topk_kernel, grid, dim3(1024), 0, st, jobs[0], jobs[n_jobs - 1], k);
        return hipGetLastError();
    }
    for (int q = 0; q < n_jobs; ++q) {
        const TopkJob &J = jobs[q];
        int64_t blocks = std::max<int64_t>(1, (n + kTopkChunk - 1) / kTopkChunk);
        // two candidate buffers of (psi, index) in turn
        const int64_t half = topk_scratch_entries(n, k) / 2;
        double *pa = (double *)J.cand, *pb = pa + half;
        int64_t *ia = (int64_t *)(pa + 2 * half), *ib = ia + half;
        hipLaunchKernelGGL(topk_level_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, st, n, k, J.stat, J.s, J.c, J.N,
                           J.w1, J.w2, J.q, (const double *)nullptr, (const int64_t *)nullptr, pa, ia);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        int64_t m = blocks * k;
        while (blocks > 1) {
            blocks = (m + kTopkChunk - 1) / kTopkChunk;
            hipLaunchKernelGGL(topk_level_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, m, k, J.stat, J.s, J.c,
                               J.N, J.w1, J.w2, J.q, pa, ia, pb, ib);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            m = blocks * k;
            std::swap(pa, pb);
            std::swap(ia, ib);
        }
        hipLaunchKernelGGL(topk_records_kernel, dim3(1), dim3(256), 0, st, k, J.stat, J.s, J.c, J.N, pa, ia, J.dec, J.out,
                           J.n_out);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Synthetic injection (Sec. 3): add amp*w_j at the template's bin, one thread
// per segment, same arithmetic as the evaluation.
__global__ __launch_bounds__(256) void inject_kernel(float *power, int n_seg, int n_bins,
                                                     int64_t k_lo, double t_sft,
                                                     const double *t_seg, const double *v,
                                                     const float *w, double f0, double tau,
                                                     double brake, double sx, double sy, double sz,
                                                     double t0, float amp,
                                                     unsigned long long *undecided) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n_seg) return;
    const double t = t_seg[j];
    if (t < t0) return;
    const double d = t - t0;
    const double qq = d / tau;
    const double u = 1.0 + qq;
    const double e = 1.0 / (1.0 - brake);
    int und = 0;
    const double g = pow_cr(u, e, &und);
    if (und) atomicAdd(undecided, 1ull);
    const double a = v[3 * j + 0] * sx;
    const double b = v[3 * j + 1] * sy;
    const double z = v[3 * j + 2] * sz;
    const double vn = (a + b) + z;
    const double D = 1.0 + vn / kC;
    const double h = g * D;
    const double H = h * t_sft;
    const double x = f0 * H;
    const double y = x + 0.5;
    const int64_t bin = (int64_t)floor(y) - k_lo;
    if (bin < 0 || bin >= n_bins) return;
    float *px = power + (int64_t)j * n_bins + bin;
    *px = *px + amp * w[j];
}

hipError_t launch_inject(float *power, int32_t n_seg, int32_t n_bins, int64_t k_lo,
                         double t_sft, const double *t_seg, const double *v, const float *w,
                         double f0, double tau, double brake, double sx, double sy, double sz,
                         double t0, float amp, unsigned long long *undecided, hipStream_t st) {
    hipLaunchKernelGGL(inject_kernel, dim3((n_seg + 255) / 256), dim3(256), 0, st, power, n_seg,
                       n_bins, k_lo, t_sft, t_seg, v, w, f0, tau, brake, sx, sy, sz, t0, amp,
                       undecided);
    return hipGetLastError();
}

}  // namespace ltgw
