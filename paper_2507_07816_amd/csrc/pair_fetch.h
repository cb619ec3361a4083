// The batches of segments that the two-realisation stack kernel fetches ahead of the
// one it sums.
#pragma once
#include "ddpow.h"

namespace ltgw {

constexpr int kPairSegs = 4, kPairAhead = 3;  // segments of a batch, batches ahead

// The first segment fetched for the batch from segment j: j, or past the last segment
// the last batch again, which nobody reads.  It is a load's scalar offset, and a
// resource's range check says nothing of one past its size; below it the product with
// the row length stays in 32 bits as well.
LTGW_HD int pair_fetch_segment(int j, int n_seg) {
    const int last = (n_seg - 1) / kPairSegs * kPairSegs;
    return j < last ? j : last;
}

}  // namespace ltgw
