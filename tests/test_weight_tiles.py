"""Which tiles a weight gradient runs in, at products whose both sides' times stand beside the rules (compiled for the host)."""
import os
import subprocess

from test_gpu_half_tiles import CUT, ROWS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HEAD = r"""
#include <cassert>
#include "routes.h"
using namespace moe;
struct Product { long M; int E, K, Nout, stream_out, accumulate, out_f32, wide_gather; };
Product product(int rows, int E, int K, int Nout, int added = 0) { return Product{(long)rows * E, E, K, Nout, (long)E * K * Nout * 2 > 48 << 20, added, added, 0}; }
"""

LINES = r"""
int main()
{
    // rows per expert, experts, K, columns, added up in fp32; tiles of 128 x 256 or of 256 x 256
    struct { int rows, E, K, Nout, added; bool half; } cases[] = {
        {4000, 1, 1056, 2080, 0, true},                                                       // a single round of the smaller ones
        {231, 6, 288, 5920, 0, true}, {364, 8, 384, 5024, 0, true}, {642, 6, 320, 5472, 0, true}, {1275, 3, 832, 5824, 0, false},  // as many rounds of either
        {22, 12, 640, 4000, 0, true}, {16, 12, 640, 4096, 0, true}, {16, 16, 544, 2752, 0, false}, {288, 12, 608, 4288, 0, false}, {143, 20, 352, 5248, 0, false},  // a third more
        {250, 8, 768, 3072, 1, true}, {482, 3, 1312, 5376, 1, true}, {822, 5, 672, 5024, 1, false}, {766, 5, 672, 5152, 1, false},  // half as many more, added to
        {250, 8, 768, 3072, 0, false}};
    for (auto& c : cases) assert(half_tiles_pay(product(c.rows, c.E, c.K, c.Nout, c.added)) == c.half);
    return 0;
}
"""


RANGES = r"""
bool behind(const Product& rows, const Product& cols) { return pair_pays(rows, 256) && !few_rows(rows) && half_round(cols); }
int main()
{
    // the layers whose ranges are tested on the device: d, h, experts, rows in all
    const long layers[][4] = {%s};
    for (auto& l : layers) {
        const int E = (int)l[2], rows = (int)(l[3] / E);
        Product by_d = product(rows, E, (int)l[0], (int)l[1]), by_h = product(rows, E, (int)l[1], (int)l[0]);
        by_d.M = by_h.M = l[3];
        // dZ (over d) beside dW2 (h high), dXs (over h) beside dW1 (d high)
        assert(behind(by_d, by_h) && behind(by_h, by_d));
        assert(half_round_slices(by_d, by_h) > 1 && half_round_slices(by_h, by_d) > 1);
    }
    // a range for each of 256 workgroups at most, and a counter and a place for each range's sum
    long cut = 0;
    for (int E : {1, 2, 3, 5, 8, 16, 40, 120, 224})
        for (int rows = 1024; rows <= 300000; rows += 1 + rows / 3)
            for (int K = 32; K <= 6000; K += 32 + K / 3)
                for (int Nout = 32; Nout <= 6000; Nout += 32 + Nout / 3) {
                    const Product cols = product(rows, E, K, Nout), dxs = product(rows, E, Nout, K);
                    if (!behind(dxs, cols)) continue;
                    const int s = half_round_slices(dxs, cols);
                    const long tiles = E * wide_columns(cols) * ((K + 127) / 128);
                    assert(s >= 1 && s <= 8 && tiles <= 256 && tiles * s <= 256);
                    cut += s > 1;
                }
    assert(cut > 100);
    return 0;
}
"""


def _run(tmp_path, program):
    (tmp_path / "tiles.cpp").write_text(HEAD + program)
    subprocess.run(["g++", "-std=c++20", "-I" + os.path.join(ROOT, "paper_2103_13262_amd", "csrc"), str(tmp_path / "tiles.cpp"), "-o", str(tmp_path / "tiles")], check=True)
    subprocess.run([str(tmp_path / "tiles")], check=True)


def test_both_sides_of_the_line(tmp_path):
    _run(tmp_path, LINES)


def test_ranges(tmp_path):
    layers = ", ".join("{%d, %d, %d, %d}" % (d, h, len(ROWS[r]), sum(ROWS[r])) for r, d, h in CUT)
    _run(tmp_path, RANGES % layers)
