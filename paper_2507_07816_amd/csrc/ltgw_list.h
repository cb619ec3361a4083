// Internal interface of the explicit-template evaluation (ltgw_list.hip) for
// the C-ABI layer.  Not part of the public boundary.
#pragma once
#include "ltgw_antenna.h"
#include "ltgw_internal.h"
#include "track_expand.h"

namespace ltgw {

// A chunk of 32 segments as the expansion kernel reads it: the time its track is
// expanded about, the largest |t_j - tc|, the smallest t_j, and the chunk's sums
// of w and w^2 in FP32, segment by segment in order.
struct ListChunk {
    double tc, dtmax, tmin;
    float w1, w2;
};

// One detector as the explicit-template kernel reads it: the store and the
// raw per-segment inputs (the tables of a lattice do not apply: every
// template has its own (tau, n) and sky direction).
struct ListDet {
    const void *store;
    int32_t pitch_bytes;
    int32_t n_seg, n_bins;
    const double *t;  // [n_seg] segment times
    const double *v;  // [n_seg][3] velocities
    const float *wq;  // [n_seg] weights x per-segment scale (the power sum)
    const float *w;   // [n_seg] weights (W1, W2)
    double t_sft, cshift;
    const double *era;     // [n_seg] Earth rotation angles, or NULL: no antenna factor
    const float *scale;    // [n_seg] store row scales (antenna weights are formed per template)
    Arms arms;
    // the expansion kernel's tables (launch_list_tables)
    const ListChunk *chunk;  // [ceil(n_seg / 32)]
    const double *dt;        // [n_seg] t_j - tc of j's chunk
    const double *vc;        // [n_seg][3] v_j / c
    const double *dop;     // [n_seg] Doppler factor 1 + v.n/c when every template has the same sky
                           // direction n (the lattice's table for it), or NULL: formed per template
};

struct ListArgs {
    ListDet det[LTGW_MAX_SEARCH_DET];
    int32_t n_det;
    double t0;
    const ltgw_template *tpl;  // [n] in the caller's order
    const int32_t *perm;       // [n] evaluation order: lane q takes template perm[q]
    int64_t n;
    double *s, *w1, *w2;       // [n] results in the caller's order
    int32_t *c, *n_in;
    float *out_s;              // optional caller outputs
    int32_t *out_c, *out_n;
    unsigned long long *in_band_total;
    unsigned long long *pow_counts;  // [0] undecided powers, [1] powers that took the double-double phase
    unsigned long long *exact_count;  // evaluations whose column the power's enclosure left open
    // expansion kernel: the chunks of all detectors in slices (slices > 1: the
    // chunk sums go to part and the counts to part_n, added by a second kernel)
    int32_t slices;
    float *part;       // [3][chunks][n]: the power sum, w and w^2 sums of each chunk
    int32_t *part_n;   // [2][slices][n]: number count, in-band segments of each slice
};

constexpr int kListChunk = 32;  // segments per chunk (the statistic's)

// The per-chunk tables of one detector; sky (3 values, or NULL) also fills dop.
hipError_t launch_list_tables(const ListDet &D, const double *sky, ListChunk *chunk, double *dt, double *vc, double *dop,
                              hipStream_t st);
// The expansion kernel: no antenna weights, and every detector with
// f0 t_sft (1 + |v|/c) < 2^19, k_lo and n_bins < 2^18 (the caller's check).
hipError_t launch_list_expansion(int store, const ListArgs &a, hipStream_t st);

hipError_t launch_template_list(int store, const ListArgs &a, hipStream_t st);

}  // namespace ltgw
