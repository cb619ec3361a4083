"""The positions of a running-median tile that each lane reads (median_slide.h, built
for the host): for every half width and for tiles of one output up to a full one, all
of them lie in the tile, every output is some lane's, and a lane that slides from one
output to the next loses and gains the positions that the two windows differ by."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_07816_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "median_slide.h"
using namespace ltgw;
int main() {
    long tiles = 0;
    for (const int N : {128, 256, 512})
    for (int h = 0; h <= 128 && 2 * h <= N - 64; ++h)
        for (int n_out = 1; n_out <= N - 2 * h; n_out += n_out < 4 || n_out + 70 > N - 2 * h ? 1 : 7) {
            const int n_pos = n_out + 2 * h, run = slide_length(n_out);
            std::vector<int> got(n_out, 0);
            for (int lane = 0; lane < 64; ++lane) {
                const SlideRun r = slide_run(lane, n_out, h);
                int leave = r.first, enter = r.enter;  // the positions of step 0
                for (int s = 0;; ++s) {
                    if (leave < 0 || leave >= n_pos || enter < 0 || enter >= n_pos) {
                        printf("h %d n_out %d lane %d step %d: reads %d and %d of %d positions\n", h, n_out, lane, s, leave,
                               enter, n_pos);
                        return 1;
                    }
                    if (r.first < 0 || r.mine < 1 || r.first + r.mine > n_out) return 2;
                    if (s < r.mine) got[r.first + s] = 1;
                    if (s + 1 == run) break;
                    if (s + 1 < r.mine && (leave != r.first + s || enter != r.first + s + 2 * h + 1)) return 3;
                    const int next = slide_next(s, r.mine);
                    leave = r.first + next;
                    enter = r.enter + next;
                }
            }
            for (int o = 0; o < n_out; ++o)
                if (!got[o]) return 4;
            ++tiles;
        }
    printf("%ld tiles\n", tiles);
    return 0;
}
"""


def test_every_position_read_is_in_the_tile(tmp_path):
    src, exe = tmp_path / "slide.cpp", tmp_path / "slide"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
