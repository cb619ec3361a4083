"""The fetches of the two-realisation stack kernel (pair_fetch.h, built for the host),
in the kernel's order: every one starts at a segment of the stack, at a byte offset below
the store's size in 32 bits, and the batch that is summed is the one it should be."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_07816_amd", "csrc")

DRIVER = r"""
#include <cstdint>
#include <cstdio>
#include "pair_fetch.h"
using namespace ltgw;
static int n_seg, set[kPairAhead], lds[2];
static int64_t pitch;
static bool issue(int q, int j) {
    const int f = pair_fetch_segment(j, n_seg);
    if (f < 0 || f >= n_seg || f * pitch >= n_seg * pitch || f * pitch > INT32_MAX) {
        printf("%d segments of %ld bytes: a fetch from segment %d\n", n_seg, (long)pitch, f);
        return false;
    }
    set[q] = f;
    return true;
}
int main() {
    for (int k = 1; k < 2000; ++k) {
        n_seg = k < 1900 ? k : (1 << 20) - (k - 1900) * 37;
        pitch = 0x7fffffffll / n_seg / 256 * 256;  // the longest row of a store below 2^31 bytes
        if (!issue(0, 0)) return 1;
        lds[0] = set[0];
        for (int q = 0; q < kPairAhead; ++q)
            if (!issue(q, (q + 1) * kPairSegs)) return 1;
        int buf = 0;
        for (int j = 0; j < n_seg;)
            for (int q = 0; q < kPairAhead; ++q)
                if (j < n_seg) {
                    if (lds[buf] != j) return 2;
                    lds[buf ^ 1] = set[q];
                    if (!issue(q, j + (kPairAhead + 1) * kPairSegs)) return 1;
                    j += kPairSegs;
                    buf ^= 1;
                }
    }
    return 0;
}
"""


def test_fetches_stay_in_the_stack(tmp_path):
    src, exe = tmp_path / "fetch.cpp", tmp_path / "fetch"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
