// Which positions of a running-median tile a lane reads as it slides over its outputs.
//
// A tile has n_out outputs and n_pos = n_out + 2 h positions, output o over positions
// o .. o + 2 h.  Lane l takes the outputs l run .. of them; lanes past the last output
// do that one again.  Between outputs the window loses position leave and gains
// position enter, both always among the tile's n_pos: a lane with one output has no
// second window, so its enter position (past the tile for the last output) is held
// at the last one, whose rank it reads and does not use.
#pragma once
#include "ddpow.h"

namespace ltgw {

struct SlideRun {
    int first;  // the lane's first output
    int mine;   // its outputs
    int enter;  // the position that its second window gains
};

// an odd run of outputs per lane (the rank reads of the lanes on different banks)
LTGW_HD int slide_length(int n_out) { return ((n_out + 63) / 64) | 1; }

LTGW_HD SlideRun slide_run(int lane, int n_out, int h) {
    const int run = slide_length(n_out), left = n_out - lane * run;
    SlideRun r;
    r.mine = left < 1 ? 1 : left < run ? left : run;
    r.first = left < 1 ? n_out - 1 : lane * run;
    const int last = n_out + 2 * h - 1, enter = r.first + 2 * h + 1;
    r.enter = enter < last ? enter : last;
    return r;
}

// the step whose positions follow those of step s (a lane that is through repeats one)
LTGW_HD int slide_next(int s, int mine) {
    const int last = mine < 2 ? 0 : mine - 2;
    return s + 1 < last ? s + 1 : last;
}

}  // namespace ltgw
