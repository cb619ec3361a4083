// Hann-windowed power spectra of strain segments, a segment per workgroup and
// nothing but the strain read and the band's powers written.
//
// A segment of N samples is M = N / 2 complex points z_n = w_2n x_2n + i w_2n+1 x_2n+1
// with M = R1 R2 R3, transformed in three register stages (n = n1 R2 R3 + n2 R3 + n3,
// k = k1 + R1 k2 + R1 R2 k3):
//   n k / M = n1 k1 / R1 + n2 k1 / (R1 R2) + n2 k2 / R2 + n3 (k1 + R1 k2) / M + n3 k3 / R3  (mod 1)
// The two exchanges between stages go through LDS, real parts and then imaginary
// parts: half the LDS, so that two workgroups of the longest segment share a CU and
// one's loads and barriers hide behind the other's arithmetic.  Row strides are padded
// so that the 64 lanes of each access fall on 64 banks.
// In the last stage a thread holds the butterflies kappa and R1 R2 - kappa, which
// are each other's mirror images: Z_k and Z_{M-k} are both in its registers, and the
// real transform's bins k and M - k follow without another exchange
// (E = (Z_k + conj Z_{M-k}) / 2, O = (Z_k - conj Z_{M-k}) / 2i, w = e^{-2 pi i k / N}:
// X_k = E + w O, X_{M-k} = conj(E - w O)).
// The window 1/2 - 1/2 cos(2 pi n / N) is applied to the samples, its cosine turned by
// the stage's constant angles from a table of one per butterfly.
//
// What bounds it is HBM: 10800 segments of 32768 samples, 8100 bins kept, 0.375 ms
// (1.77 GB at 4.7 TB/s, what a copy reaches).  hipFFT with the padding copy in
// front of it and spectra of every bin behind took 3.0 ms for the same rows.
//
// Twiddles between stages are products of two table entries (powers 4a and b of the
// thread's root): 10 loads instead of 31, one rounding more.
#include "ltgw_fft.h"

#include <utility>

namespace ltgw {

namespace {

// cos(2 pi j / 32), j = 0 .. 31
constexpr double kQ[9] = {1.0,
                          0.98078528040323044912618223613424,
                          0.92387953251128675612818318939679,
                          0.83146961230254523707878837761791,
                          0.70710678118654752440084436210485,
                          0.55557023301960222474283081394853,
                          0.38268343236508977172845998403040,
                          0.19509032201612826784828486847702,
                          0.0};
constexpr double cos32(int j) {
    j &= 31;
    if (j > 16) j = 32 - j;
    return j <= 8 ? kQ[j] : -kQ[16 - j];
}
constexpr double sin32(int j) { return cos32(j - 8); }

// register that holds output k of fft<R>
template <int R>
constexpr int at(int k) {
    if constexpr (R <= 2) return k;
    else if constexpr (R == 4) return k;
    else return (k % 4) * (R / 4) + at<R / 4>(k / 4);
}

// (re, im) *= e^{-2 pi i J / 32}
template <int J>
__device__ __forceinline__ void turn(float &re, float &im) {
    constexpr int j = J & 31;
    if constexpr (j == 0) return;
    else if constexpr (j == 8) {
        const float t = re;
        re = im;
        im = -t;
    } else if constexpr (j == 16) {
        re = -re;
        im = -im;
    } else if constexpr (j == 24) {
        const float t = re;
        re = -im;
        im = t;
    } else if constexpr (j % 8 == 4) {
        constexpr float r = (float)kQ[4];
        const float a = re, b = im;
        if constexpr (j == 4) { re = r * (a + b); im = r * (b - a); }
        else if constexpr (j == 12) { re = r * (b - a); im = -r * (a + b); }
        else if constexpr (j == 20) { re = -r * (a + b); im = r * (a - b); }
        else { re = r * (a - b); im = r * (a + b); }
    } else {
        constexpr float c = (float)cos32(j), s = (float)sin32(j);
        const float a = re, b = im;
        re = __builtin_fmaf(a, c, b * s);
        im = __builtin_fmaf(b, c, -(a * s));
    }
}

template <class F, int... I>
__device__ __forceinline__ void unroll_seq(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

template <int N, class F>
__device__ __forceinline__ void unroll(F &&f) {
    unroll_seq(f, std::make_integer_sequence<int, N>{});
}

// R-point transform in place, output k in register at<R>(k)
template <int R>
__device__ __forceinline__ void fft(float *re, float *im) {
    if constexpr (R == 2) {
        const float a = re[0], b = im[0];
        re[0] = a + re[1];
        im[0] = b + im[1];
        re[1] = a - re[1];
        im[1] = b - im[1];
    } else if constexpr (R >= 4) {
        constexpr int Q = R / 4;
        unroll<Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const float ar = re[q], ai = im[q], br = re[q + Q], bi = im[q + Q];
            const float cr = re[q + 2 * Q], ci = im[q + 2 * Q], dr = re[q + 3 * Q], di = im[q + 3 * Q];
            const float sr = ar + cr, si = ai + ci, tr = ar - cr, ti = ai - ci;
            const float ur = br + dr, ui = bi + di, vr = br - dr, vi = bi - di;
            re[q] = sr + ur;
            im[q] = si + ui;
            re[q + Q] = tr + vi;
            im[q + Q] = ti - vr;
            re[q + 2 * Q] = sr - ur;
            im[q + 2 * Q] = si - ui;
            re[q + 3 * Q] = tr - vi;
            im[q + 3 * Q] = ti + vr;
            if constexpr (Q > 1) {
                turn<q * (32 / R)>(re[q + Q], im[q + Q]);
                turn<2 * q * (32 / R)>(re[q + 2 * Q], im[q + 2 * Q]);
                turn<3 * q * (32 / R)>(re[q + 3 * Q], im[q + 3 * Q]);
            }
        });
        if constexpr (Q > 1) unroll<4>([&](auto g) { fft<Q>(re + decltype(g)::value * Q, im + decltype(g)::value * Q); });
    }
}

__device__ __forceinline__ void cmul(float &re, float &im, float2 w) {
    const float a = re, b = im;
    re = __builtin_fmaf(a, w.x, -(b * w.y));
    im = __builtin_fmaf(a, w.y, b * w.x);
}

template <int A, int B, int C>
struct Plan {
    static constexpr int R1 = A, R2 = B, R3 = C;
    static constexpr int kM = R1 * R2 * R3, kT = R1 * R2 / 2, kE = 2 * R3;
    static constexpr int kB1 = kE / R1, kB2 = kE / R2;
    static_assert(kB1 >= 1 && kB2 >= 1 && kB1 * R1 == kE && kB2 * R2 == kE && R3 >= 8 && R3 <= 16);
    static constexpr int kRow1 = R2 * R3 + R3, kRow2 = R1 * R2 + 64 / R3;
    static constexpr int kLds = R1 * kRow1 > R3 * kRow2 ? R1 * kRow1 : R3 * kRow2;
    // tables, in float2
    static constexpr int kA1 = 0;                        // [R1 / 4][R2]: W_{R1 R2}^{4 a n2}
    static constexpr int kS1 = kA1 + R1 / 4 * R2;        // [4][R2]: W_{R1 R2}^{b n2}
    static constexpr int kA2 = kS1 + 4 * R2;             // [R2 / 4][R1 R3]: W_M^{n3 (k1 + 4 a R1)}
    static constexpr int kS2 = kA2 + R2 / 4 * R1 * R3;   // [4][R3]: W_{R2 R3}^{b n3}
    static constexpr int kW = kS2 + 4 * R3;              // [R1 R2]: W_N^kappa
    static constexpr int kH = kW + R1 * R2;              // [2][R2 R3]: (cos, sin)(2 pi (2 q + e) / N) / 2
    static constexpr int kTab = kH + 2 * R2 * R3;
};

template <class P>
__global__ __launch_bounds__(256) void chip_fft_table_kernel(float2 *__restrict__ tab) {
    constexpr int R1 = P::R1, R2 = P::R2, R3 = P::R3;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= P::kTab) return;
    int64_t j, n;  // entry e^{-2 pi i j / n}
    double scale = 1.0;
    if (e < P::kS1) {
        j = (int64_t)4 * (e / R2) * (e % R2);
        n = R1 * R2;
    } else if (e < P::kA2) {
        j = (int64_t)((e - P::kS1) / R2) * ((e - P::kS1) % R2);
        n = R1 * R2;
    } else if (e < P::kS2) {
        const int p = (e - P::kA2) % (R1 * R3), a = (e - P::kA2) / (R1 * R3);
        j = (int64_t)(p % R3) * (p / R3 + 4 * a * R1);
        n = P::kM;
    } else if (e < P::kW) {
        j = (int64_t)((e - P::kS2) / R3) * ((e - P::kS2) % R3);
        n = R2 * R3;
    } else if (e < P::kH) {
        j = e - P::kW;
        n = 2 * P::kM;
    } else {
        const int q = (e - P::kH) % (R2 * R3);
        j = -(2 * q + (e - P::kH) / (R2 * R3));
        n = 2 * P::kM;
        scale = 0.5;
    }
    double s, c;
    sincospi(-2.0 * (double)j / (double)n, &s, &c);
    tab[e] = make_float2((float)(scale * c), (float)(scale * s));
}

// twiddles of one butterfly: output k times A[k / 4] S[k % 4], loaded stride apart
template <int R>
__device__ __forceinline__ void twiddle(float *re, float *im, const float2 *A, int stride_a, const float2 *S, int stride_s) {
    float2 s[4];
#pragma unroll
    for (int b = 1; b < 4; ++b) s[b] = S[b * stride_s];
    unroll<R / 4>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        const float2 w = A[a * stride_a];
        unroll<4>([&](auto bc) {
            constexpr int b = decltype(bc)::value, r = at<R>(4 * a + b);
            cmul(re[r], im[r], w);
            if constexpr (b > 0) cmul(re[r], im[r], s[b]);
        });
    });
}

template <class P>
__global__ __launch_bounds__(P::kT, 4) void chip_fft_kernel(const float2 *__restrict__ strain, int k_first, int n_out,
                                                            const float2 *__restrict__ tab, float *__restrict__ power) {
    constexpr int R1 = P::R1, R2 = P::R2, R3 = P::R3;
    constexpr int M = P::kM, T = P::kT, E = P::kE, R12 = R1 * R2;
    __shared__ float lds[P::kLds];
    const int t = threadIdx.x;
    const float2 *x = strain + (int64_t)blockIdx.x * M;
    float re[E], im[E];
    // stage 1
#pragma unroll
    for (int b = 0; b < P::kB1; ++b)
#pragma unroll
        for (int i = 0; i < R1; ++i) {
            const float2 v = x[i * (M / R1) + t + b * T];
            re[b * R1 + i] = v.x;
            im[b * R1 + i] = v.y;
        }
#pragma unroll
    for (int b = 0; b < P::kB1; ++b) {
        const int q = t + b * T;
        const float2 h0 = tab[P::kH + q], h1 = tab[P::kH + R2 * R3 + q];
        unroll<R1>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr float c = (float)cos32(i * (32 / R1)), s = (float)sin32(i * (32 / R1));
            re[b * R1 + i] *= __builtin_fmaf(h0.y, s, __builtin_fmaf(-h0.x, c, 0.5f));
            im[b * R1 + i] *= __builtin_fmaf(h1.y, s, __builtin_fmaf(-h1.x, c, 0.5f));
        });
        fft<R1>(re + b * R1, im + b * R1);
        twiddle<R1>(re + b * R1, im + b * R1, tab + P::kA1 + q / R3, R2, tab + P::kS1 + q / R3, R2);
    }
    // exchange 1: rows k1 of R2 R3 + R3
    auto put1 = [&](const float *v) {
#pragma unroll
        for (int b = 0; b < P::kB1; ++b)
            unroll<R1>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                lds[k * P::kRow1 + t + b * T] = v[b * R1 + at<R1>(k)];
            });
    };
    auto get1 = [&](float *v) {
#pragma unroll
        for (int b = 0; b < P::kB2; ++b) {
            const int p = t + b * T;
#pragma unroll
            for (int i = 0; i < R2; ++i) v[b * R2 + i] = lds[p / R3 * P::kRow1 + i * R3 + p % R3];
        }
    };
    put1(re);
    __syncthreads();
    get1(re);
    __syncthreads();
    put1(im);
    __syncthreads();
    get1(im);
    // stage 2
#pragma unroll
    for (int b = 0; b < P::kB2; ++b) {
        const int p = t + b * T;
        fft<R2>(re + b * R2, im + b * R2);
        twiddle<R2>(re + b * R2, im + b * R2, tab + P::kA2 + p, R1 * R3, tab + P::kS2 + p % R3, R3);
    }
    // exchange 2: rows n3 of R1 R2 + 64 / R3
    auto put2 = [&](const float *v) {
#pragma unroll
        for (int b = 0; b < P::kB2; ++b) {
            const int p = t + b * T;
            unroll<R2>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                lds[p % R3 * P::kRow2 + p / R3 + R1 * k] = v[b * R2 + at<R2>(k)];
            });
        }
    };
    const int kb = t ? R12 - t : R12 / 2;  // the second butterfly's kappa
    auto get2 = [&](float *v) {
#pragma unroll
        for (int i = 0; i < R3; ++i) {
            v[i] = lds[i * P::kRow2 + t];
            v[R3 + i] = lds[i * P::kRow2 + kb];
        }
    };
    __syncthreads();
    put2(re);
    __syncthreads();
    get2(re);
    __syncthreads();
    put2(im);
    __syncthreads();
    get2(im);
    // stage 3
    fft<R3>(re, im);
    fft<R3>(re + R3, im + R3);
    float *out = power + (int64_t)blockIdx.x * n_out;
    // bins k and M - k from Z_k (registers a) and Z_{M-k} (registers m); w = W_N^k
    auto bins = [&](int k, int a, int m, float wr, float wi) {
        const int o0 = k - k_first, o1 = M - k - k_first;
        const bool in0 = (unsigned)o0 < (unsigned)n_out, in1 = (unsigned)o1 < (unsigned)n_out;
        if (!(in0 || in1)) return;
        const float er = 0.5f * (re[a] + re[m]), ei = 0.5f * (im[a] - im[m]);
        float vr = 0.5f * (im[a] + im[m]), vi = 0.5f * (re[m] - re[a]);
        cmul(vr, vi, make_float2(wr, wi));
        const float pr = er + vr, pi = ei + vi, qr = er - vr, qi = ei - vi;
        if (in0) out[o0] = __builtin_fmaf(pr, pr, pi * pi);
        if (in1) out[o1] = __builtin_fmaf(qr, qr, qi * qi);
    };
    const float2 wk = tab[P::kW + t];
    if (t) {
        unroll<R3>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            float wr = wk.x, wi = wk.y;
            turn<k * (16 / R3)>(wr, wi);
            bins(t + R12 * k, at<R3>(k), R3 + at<R3>(R3 - 1 - k), wr, wi);
        });
    } else {  // kappa = 0 and R1 R2 / 2 are their own mirror images
        unroll<R3 / 2 + 1>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            float wr = 1.0f, wi = 0.0f;
            turn<k * (16 / R3)>(wr, wi);
            bins(R12 * k, at<R3>(k), at<R3>((R3 - k) % R3), wr, wi);
        });
        const float2 wh = tab[P::kW + R12 / 2];
        unroll<R3 / 2>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            float wr = wh.x, wi = wh.y;
            turn<k * (16 / R3)>(wr, wi);
            bins(R12 / 2 + R12 * k, R3 + at<R3>(k), R3 + at<R3>(R3 - 1 - k), wr, wi);
        });
    }
}

// f(plan) for a supported n_fft
template <class F>
bool with_plan(int32_t n_fft, F &&f) {
    switch (n_fft) {
        case 4096: f(Plan<16, 16, 8>{}); return true;
        case 8192: f(Plan<16, 16, 16>{}); return true;
        case 16384: f(Plan<32, 16, 16>{}); return true;
        case 32768: f(Plan<32, 32, 16>{}); return true;
        default: return false;
    }
}

}  // namespace

bool chip_fft_has(int32_t n_fft) {
    return with_plan(n_fft, [](auto) {});
}

size_t chip_fft_table_bytes(int32_t n_fft) {
    size_t n = 0;
    with_plan(n_fft, [&](auto p) { n = decltype(p)::kTab * sizeof(float2); });
    return n;
}

hipError_t launch_chip_fft_tables(int32_t n_fft, float2 *tab, hipStream_t st) {
    if (!with_plan(n_fft, [&](auto p) {
            using P = decltype(p);
            hipLaunchKernelGGL(chip_fft_table_kernel<P>, dim3((P::kTab + 255) / 256), dim3(256), 0, st, tab);
        }))
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_chip_fft(int32_t n_fft, const float *strain, int32_t n_seg, int64_t k_first, int32_t n_out,
                           const float2 *tab, float *power, hipStream_t st) {
    if (!with_plan(n_fft, [&](auto p) {
            using P = decltype(p);
            hipLaunchKernelGGL(chip_fft_kernel<P>, dim3((unsigned)n_seg), dim3(P::kT), 0, st, (const float2 *)strain,
                               (int)k_first, n_out, tab, power);
        }))
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace ltgw
