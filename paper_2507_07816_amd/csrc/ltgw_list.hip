// The statistic of an explicit template list: the uniform random template
// bank of Sec. 2, where every template has its own (f0, tau, n, sky) and no
// per-group table can be shared.
#include "ltgw_gather.h"
#include "ltgw_list.h"
#include "ddpow.h"
#include "pow_enclose.h"

#pragma clang fp contract(off)

namespace ltgw {

// segments whose columns and gathers are formed together (divides kChunk)
constexpr int kListBatch = 8;
static_assert(kChunk % kListBatch == 0, "a batch must not straddle a chunk");

// D_j = 1 + v_j.n/c (Eq. 2): the detector's table for a one-sky list, else
// formed from the template's sky direction
template <bool DOP>
__device__ inline double doppler(const ListDet &D, int j, const ltgw_template &T) {
    if (DOP) return uniform_load(D.dop, j);
    const double va = uniform_load(D.v, 3 * j + 0) * T.sky[0];
    const double vb = uniform_load(D.v, 3 * j + 1) * T.sky[1];
    const double vz = uniform_load(D.v, 3 * j + 2) * T.sky[2];
    const double vn = (va + vb) + vz;
    return 1.0 + div_rn(vn, kC, kInvC);
}

// The enclosure's tables as copies in LDS (filled once per workgroup): a
// wavefront's 64 lanes read scattered entries, which LDS serves in a few
// cycles where the constant arrays cost a round trip through the cache.
struct LdsTables {
    const double2 *lg;  // [128] (r_i, RN(-log r_i))
    const double *ex;   // [256] RN(2^(j/256))
    __device__ void log_entry(int i, double *r, double *t) const {
        const double2 v = lg[i];
        *r = v.x;
        *t = v.y;
    }
    __device__ double exp2_entry(int j) const { return ex[j]; }
};

// the column of the track for spin-down factor g; monotone in g
__device__ inline unsigned column(const ListDet &D, const ltgw_template &T, double Df, double g) {
    const double h = g * Df;
    const double H = h * D.t_sft;
    const double x = T.f0 * H;
    return (unsigned)__double2int_rz(x + D.cshift);
}

// Lane q evaluates template perm[q] over every selected detector and segment
// with the lattice's arithmetic, in its order:
//   t < T0: masked (g = 0, so the column falls out of band)
//   u = 1 + (t - T0)/tau, e = 1/(1 - n), g = RN(u^e)            (Eq. 1)
//   D = 1 + ((vx nx + vy ny) + vz nz)/c, H = RN(RN(g D) T_sft)   (Eq. 2)
//   x = f0 H, column = trunc(x + 1.5 - k_lo), gather, FP32 sums over chunks
//   of 32 segments carried in FP64                               (Sec. 2)
// so a template of a lattice gets that lattice's s, c and N bit for bit (the
// two quotients come from reciprocals by div_rn, which equals the division).
// The column is monotone in g, so it is taken at both ends of a cheap
// enclosure of RN(u^e) (pow_enclose.h); only where they differ (about one
// evaluation in 10^8, counted) is RN(u^e) itself evaluated, by the
// double-double power (its decisions are those of the two-phase power that
// fills a lattice's table wherever it decides).  That call stays out of line,
// so the kernel holds only the enclosure's registers.
// Segments go in batches of SB: the enclosure runs stage by stage over the
// batch (all its log-table reads, then all its exp-table reads, from copies
// of the tables in LDS), the batch's gathers are issued together, and the
// sums are taken in segment order, as one segment at a time would.  Without
// the batches each segment's chain of dependent reads ran alone.  Sorting the
// list by f0 (the caller's perm) keeps neighbouring lanes on neighbouring
// columns for the gathers.
// ANT: some detector carries antenna-pattern weights.  Without, the kernel
// holds none of their per-detector values, which leaves the scalar registers
// to the power's constants (else they spill into vector-register lanes).
// DOP: every detector has a Doppler table (one sky direction for the whole
// list), read per segment instead of formed per template.
template <int STORE, bool ANT, bool DOP, int SB>
__global__ __launch_bounds__(256) void template_list_kernel(const ListArgs a) {
    __shared__ double2 s_log[128];
    __shared__ double s_exp[256];
    {
        const EncloseTables ct;
        if (threadIdx.x < 128) {
            double r, t;
            ct.log_entry(threadIdx.x, &r, &t);
            s_log[threadIdx.x] = make_double2(r, t);
        }
        s_exp[threadIdx.x] = ct.exp2_entry(threadIdx.x);
        __syncthreads();
    }
    const LdsTables tab{s_log, s_exp};
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool live = q < a.n;
    // lanes past the list evaluate its first template and discard it; they
    // take no correctly rounded power and count nothing
    const int32_t o = live ? a.perm[q] : a.perm[0];
    const ltgw_template T = a.tpl[o];
    const double e = 1.0 / (1.0 - T.brake);
    const double rtau = 1.0 / T.tau;  // RN(1/tau): the per-segment quotients by div_rn
    double s = 0.0, w1 = 0.0, w2 = 0.0;
    int cnt = 0, nin = 0;
    for (int d = 0; d < a.n_det; ++d) {
        const ListDet D = a.det[d];
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void *)D.store, Store<STORE>::kBytes, D.n_bins + 2, kBufDword3);
        const unsigned nb = (unsigned)D.n_bins;
        for (int j0 = 0; j0 < D.n_seg; j0 += kChunk) {
            const int je = min(j0 + kChunk, D.n_seg);
            float sc = 0.0f, w1c = 0.0f, w2c = 0.0f;
            for (int jb = j0; jb < je; jb += SB) {
                unsigned idx[SB];
                unsigned open = 0;  // bit b: segment jb + b needs RN(u^e) itself
                EncloseSplit sp[SB];
#pragma unroll
                for (int b = 0; b < SB; ++b) {
                    const double t = uniform_load(D.t, min(jb + b, je - 1));
                    sp[b] = enclose_split(1.0 + div_rn(t - a.t0, T.tau, rtau));
                }
                double ri[SB], ti[SB];
#pragma unroll
                for (int b = 0; b < SB; ++b) tab.log_entry(sp[b].i, &ri[b], &ti[b]);
                EncloseLog lg[SB];
                double x2[SB];
#pragma unroll
                for (int b = 0; b < SB; ++b) lg[b] = enclose_log(e, sp[b], ri[b], ti[b]);
#pragma unroll
                for (int b = 0; b < SB; ++b) x2[b] = tab.exp2_entry(lg[b].j);
#pragma unroll
                for (int b = 0; b < SB; ++b) {
                    const int j = min(jb + b, je - 1);
                    const double Df = doppler<DOP>(D, j, T);
                    const bool before = uniform_load(D.t, j) < a.t0;  // masked: g = 0
                    double glo, ghi;
                    enclose_ends(enclose_value(lg[b], x2[b]), lg[b].y, e, &glo, &ghi);
                    idx[b] = column(D, T, Df, before ? 0.0 : glo);
                    const bool decided = before || (lg[b].ok && column(D, T, Df, ghi) == idx[b]);
                    if (!decided && jb + b < je && live) open |= 1u << b;
                }
                if (open) {
                    for (int b = 0; b < SB; ++b) {
                        if (!((open >> b) & 1u)) continue;
                        const int j = jb + b;
                        const double u = 1.0 + div_rn(uniform_load(D.t, j) - a.t0, T.tau, rtau);
                        const PowSlow px = pow_dd_call(u, e);
                        idx[b] = column(D, T, doppler<DOP>(D, j, T), px.g);
                        atomicAdd(a.exact_count, 1ull);
                        atomicAdd(a.pow_counts + 1, 1ull);
                        if (px.undecided) atomicAdd(a.pow_counts, 1ull);
                    }
                }
                float p[SB];
#pragma unroll
                for (int b = 0; b < SB; ++b)
                    p[b] = jb + b < je ? Store<STORE>::get(rs, (int)idx[b], (jb + b) * D.pitch_bytes, cnt) : 0.0f;
#pragma unroll
                for (int b = 0; b < SB; ++b) {
                    if (jb + b >= je) break;
                    const int j = jb + b;
                    float wq = uniform_load(D.wq, j), wv = uniform_load(D.w, j);
                    if (ANT && D.era)  // antenna-pattern weights for this template's sky direction
                        antenna_weights(D.arms, uniform_load(D.era, j), T.sky[0], T.sky[1], T.sky[2], wv,
                                        uniform_load(D.scale, j), wv, wq);
                    sc = __builtin_fmaf(wq, p[b], sc);
                    const bool inb = (idx[b] - 1u) < nb;
                    nin += inb ? 1 : 0;
                    const float wj = inb ? wv : 0.0f;
                    w1c += wj;
                    w2c = __builtin_fmaf(wj, wj, w2c);
                }
            }
            s += (double)sc;
            w1 += (double)w1c;
            w2 += (double)w2c;
        }
    }
    // the in-band total of the list (diagnostics): one atomic per wavefront
    unsigned long long mine = live ? (unsigned long long)nin : 0ull;
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(a.in_band_total, mine);
    if (!live) return;
    a.s[o] = s;
    a.c[o] = cnt;
    a.n_in[o] = nin;
    a.w1[o] = w1;
    a.w2[o] = w2;
    if (a.out_s) a.out_s[o] = (float)s;
    if (a.out_c) a.out_c[o] = cnt;
    if (a.out_n) a.out_n[o] = nin;
}

// ---------------------------------------------------------------------------
// The same evaluation with a template's track expanded about the middle of each
// chunk of 32 segments (track_expand.h): one enclosure value per chunk and a
// degree-6 polynomial per segment in place of a logarithm and an exponential.
// Where the series leaves a column open, the evaluation is decided as before, by the
// enclosure of RN(u^e) and, failing that, by RN(u^e) itself, so every column is the
// contract's.  A chunk goes that way segment by segment where the series does
// not hold (a large step against tau) or a segment lies before T0.
//
// W1, W2 and N need no work per segment where a lane is in band throughout a
// chunk (the chunk's sums of w and w^2, the same in every lane) or out of band
// throughout; other lanes take the chunk's segments again.
//
// A list too short to fill the chip is split over its chunks (blockIdx.y): each
// slice writes its FP32 chunk sums, and list_reduce_kernel adds them per template
// in segment order, the FP64 operations of the unsplit sum.
//
// 10^6 templates x 10800 segments: 47.7 -> 11.7 ms (2.3e11 -> 9.2e11 evaluations/s);
// 4800 x 1024: 637 -> 36 + 6 us, one chunk per workgroup.
// RN-chain column of one evaluation, out of line: the enclosure and, where it
// stays open, the double-double power.
struct ListColumn {
    unsigned idx;
    int exact, undecided;
};
__device__ __attribute__((noinline)) ListColumn list_column(double dt0, double tau, double rtau, double e, double Df,
                                                            double t_sft, double f0, double cshift) {
    auto col = [&](double g) {
        const double h = g * Df;
        const double H = h * t_sft;
        const double x = f0 * H;
        return (unsigned)__double2int_rz(x + cshift);
    };
    ListColumn r{0u, 0, 0};
    if (dt0 < 0.0) {  // before T0: masked, g = 0
        r.idx = col(0.0);
        return r;
    }
    const double u = 1.0 + div_rn(dt0, tau, rtau);
    double lo, hi;
    if (pow_enclose(u, e, &lo, &hi)) {
        r.idx = col(lo);
        if (col(hi) == r.idx) return r;
    }
    const PowSlow px = pow_dd_call(u, e);
    r.idx = col(px.g);
    r.exact = 1;
    r.undecided = px.undecided;
    return r;
}

template <bool DOP>
__device__ inline double list_doppler(const ListDet &D, int j, const ltgw_template &T) {
    if (DOP) return uniform_load(D.dop, j);
    // within 2^-51 of Eq. 2's chain: the margin covers it
    double d = __builtin_fma(uniform_load(D.vc, 3 * j + 2), T.sky[2], 1.0);
    d = __builtin_fma(uniform_load(D.vc, 3 * j + 1), T.sky[1], d);
    return __builtin_fma(uniform_load(D.vc, 3 * j + 0), T.sky[0], d);
}

template <int STORE, bool DOP, bool SPLIT>
__global__ __launch_bounds__(256) void list_expansion_kernel(const ListArgs a, int total_chunks) {
    __shared__ double2 s_log[128];
    __shared__ double s_exp[256];
    {
        const EncloseTables ct;
        if (threadIdx.x < 128) {
            double r, t;
            ct.log_entry(threadIdx.x, &r, &t);
            s_log[threadIdx.x] = make_double2(r, t);
        }
        s_exp[threadIdx.x] = ct.exp2_entry(threadIdx.x);
        __syncthreads();
    }
    const LdsTables tab{s_log, s_exp};
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool live = q < a.n;
    // lanes past the list evaluate its first template and discard it
    const int32_t o = live ? a.perm[q] : a.perm[0];
    const ltgw_template T = a.tpl[o];
    const double e = 1.0 / (1.0 - T.brake);
    const double rtau = 1.0 / T.tau;
    double c[7];
    expand_series(e, c);
    const int g0 = SPLIT ? (int)((int64_t)total_chunks * blockIdx.y / gridDim.y) : 0;
    const int g1 = SPLIT ? (int)((int64_t)total_chunks * (blockIdx.y + 1) / gridDim.y) : total_chunks;
    double s = 0.0, w1 = 0.0, w2 = 0.0;
    int cnt = 0, nin = 0;
    int first = 0;  // the detector's first chunk in the list of all
    for (int d = 0; d < a.n_det; ++d) {
        const ListDet D = a.det[d];
        const int nch = (D.n_seg + kChunk - 1) / kChunk;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void *)D.store, Store<STORE>::kBytes, D.n_bins + 2, kBufDword3);
        const unsigned nb = (unsigned)D.n_bins;
        const double f0T = T.f0 * D.t_sft;
        const double M = 0x1p20 + D.cshift;
        const int c_end = min(nch, g1 - first);
        for (int ch = max(0, g0 - first); ch < c_end; ++ch) {
            const int j0 = ch * kChunk, nj = min(kChunk, D.n_seg - j0);
            const double tc = uniform_load(&D.chunk[ch].tc, 0), dtmax = uniform_load(&D.chunk[ch].dtmax, 0);
            const double tau_c = T.tau + (tc - a.t0);
            const double r = 1.0 / tau_c;
            const EncloseSplit sp = enclose_split(tau_c * rtau);
            double ri, ti;
            tab.log_entry(sp.i, &ri, &ti);
            const EncloseLog lg = enclose_log(e, sp, ri, ti);
            const double A = f0T * enclose_value(lg, tab.exp2_entry(lg.j));
            const double dm = dtmax * r;
            const double m = expand_margin(A, dm, c[6], lg.y, e);
            const bool fast = (lg.ok && expand_holds(dm, m, e)) || !live;
            const bool masked = uniform_load(&D.chunk[ch].tmin, 0) < a.t0;
            // the column of segment j by the contract's chain
            auto exact_column = [&](int j, bool count) -> unsigned {
                double Df;
                if (DOP) {
                    Df = uniform_load(D.dop, j);
                } else {
                    Df = doppler<false>(D, j, T);
                }
                const ListColumn k = list_column(uniform_load(D.t, j) - a.t0, T.tau, rtau, e, Df, D.t_sft, T.f0, D.cshift);
                if (k.exact && count) {
                    atomicAdd(a.exact_count, 1ull);
                    atomicAdd(a.pow_counts + 1, 1ull);
                    if (k.undecided) atomicAdd(a.pow_counts, 1ull);
                }
                return k.idx;
            };
            float sc = 0.0f, w1c = 0.0f, w2c = 0.0f;
            if (!masked && __all(fast)) {
                const unsigned mi = expand_margin_units(m);
                double k[7];
                k[0] = A;
#pragma unroll
                for (int i = 0; i < 6; ++i) k[i + 1] = A * c[i];
                auto fast_column = [&](int j, unsigned &z) -> unsigned {
                    return expand_column(expand_x(k, uniform_load(D.dt, j) * r, list_doppler<DOP>(D, j, T)), M, mi, &z);
                };
                unsigned bits = 0, lo = ~0u, hi = 0u;
                for (int jb = 0; jb < nj; jb += kListBatch) {
                    unsigned idx[kListBatch], z[kListBatch];
#pragma unroll
                    for (int b = 0; b < kListBatch; ++b) idx[b] = fast_column(j0 + min(jb + b, nj - 1), z[b]);
                    unsigned zm = z[0];
#pragma unroll
                    for (int b = 1; b < kListBatch; ++b) zm = min(zm, z[b]);
                    if (zm < 2u * mi && live) {
#pragma unroll 1
                        for (int b = 0; b < kListBatch; ++b) {
                            unsigned zz;
                            const int j = j0 + min(jb + b, nj - 1);
                            unsigned v = fast_column(j, zz);
                            if (zz < 2u * mi) v = exact_column(j, jb + b < nj);
#pragma unroll
                            for (int u = 0; u < kListBatch; ++u) idx[u] = u == b ? v : idx[u];
                        }
                    }
                    float p[kListBatch];
#pragma unroll
                    for (int b = 0; b < kListBatch; ++b)
                        p[b] = Store<STORE>::load(rs, (int)idx[b], (j0 + min(jb + b, nj - 1)) * D.pitch_bytes);
                    // a power that BF16 rounded to infinity is not to meet the weight 0 of a
                    // segment past the last (the other stores hold finite values)
                    if (STORE == LTGW_STORE_BF16 && jb + kListBatch > nj)
#pragma unroll
                        for (int b = 0; b < kListBatch; ++b) p[b] = jb + b < nj ? p[b] : 0.0f;
#pragma unroll
                    for (int b = 0; b < kListBatch; ++b) {
                        // a segment past the last has weight 0 and its count bit is shifted out below
                        const float wq = jb + b < nj ? uniform_load(D.wq, j0 + min(jb + b, nj - 1)) : 0.0f;
                        sc = __builtin_fmaf(wq, __builtin_fabsf(p[b]), sc);
                        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(p[b]), 31);
                        lo = min(lo, idx[b]);
                        hi = max(hi, idx[b]);
                    }
                }
                const int done = (nj + kListBatch - 1) / kListBatch * kListBatch;
                cnt += __popc(bits >> (done - nj));
                const bool all_in = lo >= 1u && hi <= nb, all_out = lo > nb;
                if (all_in) {
                    w1c = uniform_load(&D.chunk[ch].w1, 0);
                    w2c = uniform_load(&D.chunk[ch].w2, 0);
                    nin += nj;
                }
                if (!all_in && !all_out) {
#pragma unroll 1
                    for (int j = j0; j < j0 + nj; ++j) {
                        unsigned z;
                        unsigned v = fast_column(j, z);
                        if (z < 2u * mi) v = exact_column(j, false);
                        const bool inb = (v - 1u) < nb;
                        nin += inb ? 1 : 0;
                        const float wj = inb ? uniform_load(D.w, j) : 0.0f;
                        w1c += wj;
                        w2c = __builtin_fmaf(wj, wj, w2c);
                    }
                }
            } else {
#pragma unroll 1
                for (int j = j0; j < j0 + nj; ++j) {
                    const unsigned v = exact_column(j, live);
                    const float p = Store<STORE>::load(rs, (int)v, j * D.pitch_bytes);
                    sc = __builtin_fmaf(uniform_load(D.wq, j), __builtin_fabsf(p), sc);
                    cnt += (int)(__float_as_uint(p) >> 31);
                    const bool inb = (v - 1u) < nb;
                    nin += inb ? 1 : 0;
                    const float wj = inb ? uniform_load(D.w, j) : 0.0f;
                    w1c += wj;
                    w2c = __builtin_fmaf(wj, wj, w2c);
                }
            }
            if (SPLIT) {
                if (live) {
                    float *p = a.part + (int64_t)(first + ch) * a.n + q;
                    p[0] = sc;
                    p[(int64_t)total_chunks * a.n] = w1c;
                    p[2 * (int64_t)total_chunks * a.n] = w2c;
                }
            } else {
                s += (double)sc;
                w1 += (double)w1c;
                w2 += (double)w2c;
            }
        }
        first += nch;
    }
    // the in-band total of the list (diagnostics): one atomic per wavefront
    unsigned long long mine = live ? (unsigned long long)nin : 0ull;
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(a.in_band_total, mine);
    if (!live) return;
    if (SPLIT) {
        a.part_n[(int64_t)blockIdx.y * a.n + q] = cnt;
        a.part_n[((int64_t)gridDim.y + blockIdx.y) * a.n + q] = nin;
        return;
    }
    a.s[o] = s;
    a.c[o] = cnt;
    a.n_in[o] = nin;
    a.w1[o] = w1;
    a.w2[o] = w2;
    if (a.out_s) a.out_s[o] = (float)s;
    if (a.out_c) a.out_c[o] = cnt;
    if (a.out_n) a.out_n[o] = nin;
}

// The sums of a split list: per template its chunk sums in segment order.
__global__ __launch_bounds__(64) void list_reduce_kernel(const ListArgs a, int total_chunks) {
    const int64_t q = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (q >= a.n) return;
    const int32_t o = a.perm[q];
    double s = 0.0, w1 = 0.0, w2 = 0.0;
    const float *p = a.part + q;
    const int64_t st = (int64_t)total_chunks * a.n;
#pragma unroll 8
    for (int ch = 0; ch < total_chunks; ++ch) {
        s += (double)p[ch * a.n];
        w1 += (double)p[st + ch * a.n];
        w2 += (double)p[2 * st + ch * a.n];
    }
    int cnt = 0, nin = 0;
#pragma unroll 8
    for (int k = 0; k < a.slices; ++k) {
        cnt += a.part_n[(int64_t)k * a.n + q];
        nin += a.part_n[((int64_t)a.slices + k) * a.n + q];
    }
    a.s[o] = s;
    a.c[o] = cnt;
    a.n_in[o] = nin;
    a.w1[o] = w1;
    a.w2[o] = w2;
    if (a.out_s) a.out_s[o] = (float)s;
    if (a.out_c) a.out_c[o] = cnt;
    if (a.out_n) a.out_n[o] = nin;
}

template <int STORE, bool DOP>
static void launch_expansion_store(const ListArgs &a, int chunks, hipStream_t st) {
    const dim3 grid((unsigned)((a.n + 255) / 256), (unsigned)a.slices);
    if (a.slices > 1)
        hipLaunchKernelGGL((list_expansion_kernel<STORE, DOP, true>), grid, dim3(256), 0, st, a, chunks);
    else
        hipLaunchKernelGGL((list_expansion_kernel<STORE, DOP, false>), grid, dim3(256), 0, st, a, chunks);
}

hipError_t launch_list_expansion(int store, const ListArgs &a, hipStream_t st) {
    if (a.n < 1 || a.n > 0x7fffffffLL || a.slices < 1 || a.slices > 65535) return hipErrorInvalidValue;
    bool dop = true;
    int chunks = 0;
    for (int d = 0; d < a.n_det; ++d) {
        dop = dop && a.det[d].dop != nullptr;
        chunks += (a.det[d].n_seg + kChunk - 1) / kChunk;
    }
    if (a.slices > 1 && (!a.part || !a.part_n)) return hipErrorInvalidValue;
#define LTGW_EXPANSION(S)                              \
    if (dop)                                           \
        launch_expansion_store<S, true>(a, chunks, st); \
    else                                               \
        launch_expansion_store<S, false>(a, chunks, st)
    if (store == LTGW_STORE_F32) {
        LTGW_EXPANSION(LTGW_STORE_F32);
    } else if (store == LTGW_STORE_BF16) {
        LTGW_EXPANSION(LTGW_STORE_BF16);
    } else {
        LTGW_EXPANSION(LTGW_STORE_FP8);
    }
#undef LTGW_EXPANSION
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.slices == 1) return e;
    hipLaunchKernelGGL(list_reduce_kernel, dim3((unsigned)((a.n + 63) / 64)), dim3(64), 0, st, a, chunks);
    return hipGetLastError();
}

// The tables of one detector: 8 chunks per workgroup, a lane per segment; the
// first lane of each chunk forms its sums in order.
__global__ __launch_bounds__(256) void list_tables_kernel(const ListDet D, int with_sky, double sx, double sy, double sz,
                                                          ListChunk *__restrict__ chunk, double *__restrict__ dt,
                                                          double *__restrict__ vc, double *__restrict__ dop) {
    __shared__ double st[256];
    __shared__ float sw[256];
    const int j = blockIdx.x * 256 + (int)threadIdx.x;
    const int lead = (int)threadIdx.x & ~(kChunk - 1);
    const bool in = j < D.n_seg;
    st[threadIdx.x] = in ? D.t[j] : 0.0;
    sw[threadIdx.x] = in ? D.w[j] : 0.0f;
    __syncthreads();
    const int nj = min(kChunk, D.n_seg - (int)(blockIdx.x * 256) - lead);
    if (nj <= 0) return;
    const double tc = st[lead + nj / 2];
    if (in) {
        dt[j] = st[threadIdx.x] - tc;
        double va[3];
        for (int k = 0; k < 3; ++k) {
            va[k] = D.v[3 * j + k];
            vc[3 * j + k] = va[k] / kC;
        }
        if (with_sky) {  // the lattice's operations in its order (doppler_kernel)
            const double vx = va[0] * sx, vy = va[1] * sy, vz = va[2] * sz;
            const double vn = (vx + vy) + vz;
            const double r = vn / kC;
            dop[j] = 1.0 + r;
        }
    }
    if ((int)threadIdx.x != lead) return;
    ListChunk c;
    c.tc = tc;
    c.dtmax = 0.0;
    c.tmin = tc;
    c.w1 = c.w2 = 0.0f;
    for (int k = 0; k < nj; ++k) {
        c.dtmax = fmax(c.dtmax, fabs(st[lead + k] - tc));
        c.tmin = fmin(c.tmin, st[lead + k]);
        c.w1 += sw[lead + k];
        c.w2 = __builtin_fmaf(sw[lead + k], sw[lead + k], c.w2);
    }
    chunk[j / kChunk] = c;
}

hipError_t launch_list_tables(const ListDet &D, const double *sky, ListChunk *chunk, double *dt, double *vc, double *dop,
                              hipStream_t st) {
    hipLaunchKernelGGL(list_tables_kernel, dim3((unsigned)((D.n_seg + 255) / 256)), dim3(256), 0, st, D, sky ? 1 : 0,
                       sky ? sky[0] : 0.0, sky ? sky[1] : 0.0, sky ? sky[2] : 0.0, chunk, dt, vc, dop);
    return hipGetLastError();
}

template <int STORE>
static void launch_list_store(bool ant, bool dop, const ListArgs &a, dim3 grid, hipStream_t st) {
    if (ant)
        hipLaunchKernelGGL((template_list_kernel<STORE, true, false, kListBatch>), grid, dim3(256), 0, st, a);
    else if (dop)
        hipLaunchKernelGGL((template_list_kernel<STORE, false, true, kListBatch>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((template_list_kernel<STORE, false, false, kListBatch>), grid, dim3(256), 0, st, a);
}

hipError_t launch_template_list(int store, const ListArgs &a, hipStream_t st) {
    if (a.n < 1 || a.n > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((a.n + 255) / 256));
    bool ant = false, dop = true;
    for (int d = 0; d < a.n_det; ++d) {
        ant = ant || a.det[d].era != nullptr;
        dop = dop && a.det[d].dop != nullptr;
    }
    if (store == LTGW_STORE_F32)
        launch_list_store<LTGW_STORE_F32>(ant, dop, a, grid, st);
    else if (store == LTGW_STORE_BF16)
        launch_list_store<LTGW_STORE_BF16>(ant, dop, a, grid, st);
    else
        launch_list_store<LTGW_STORE_FP8>(ant, dop, a, grid, st);
    return hipGetLastError();
}

}  // namespace ltgw
