"""Which kernel a bf16 product runs in, at layers whose both sides' times stand beside the rules (compiled for the host)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cassert>
#include "routes.h"
using namespace moe;
struct Product { long M; int E, K, Nout, stream_out, accumulate, out_f32, wide_gather; };
Product product(int rows, int E, int K, int Nout) { return Product{(long)rows * E, E, K, Nout, (long)E * K * Nout * 2 > 48 << 20, 0, 0, 0}; }

int main()
{
    // rows per expert, experts, reduction, columns
    struct { int rows, E, K, Nout; bool small; } forward[] = {
        {8, 16, 1024, 4096, true}, {64, 256, 512, 1024, true}, {95, 4, 4096, 4096, true},
        {250, 8, 768, 3072, true}, {250, 8, 3072, 768, true}, {430, 5, 800, 2112, true}, {512, 16, 1024, 4096, false}, {512, 16, 4096, 1024, false},
        {226, 6, 7712, 3712, false}, {5223, 1, 7104, 896, true}, {4568, 1, 6496, 1088, false},                     // deep
        {8192, 1, 512, 2048, false}, {8192, 1, 4096, 1024, false}, {1705, 2, 896, 3488, false}, {2048, 1, 1024, 4096, true}, {1532, 2, 512, 768, true},   // whole blocks
        {290, 222, 1088, 384, true}, {1498, 9, 5056, 800, false}, {476, 64, 4512, 288, true}, {1630, 18, 7584, 352, false}};   // columns that are not there
    for (auto& c : forward) assert(route(product(c.rows, c.E, c.K, c.Nout), true) == (c.small ? Route::kSmallTiles : Route::kClasses));
    struct { int rows, E, K, Nout; Route to; } backward[] = {
        {61, 111, 1408, 2144, Route::kSmallTiles}, {64, 64, 1024, 2048, Route::kTiles64}, {34, 97, 1024, 544, Route::kSmallTiles},
        {250, 8, 3072, 768, Route::kSmallTiles}, {90, 7, 2432, 320, Route::kSmallTiles}, {512, 16, 4096, 1024, Route::kClasses},
        {4096, 1, 4096, 1024, Route::kClasses}, {2048, 2, 2048, 1024, Route::kClasses}, {2048, 1, 8192, 2048, Route::kSmallTiles}};
    for (auto& c : backward) assert(route(product(c.rows, c.E, c.K, c.Nout), false) == c.to);
    // a pair never holds a product that runs in small tiles, or operands beyond 32-bit offsets
    for (auto& c : backward) {
        Product p = product(c.rows, c.E, c.K, c.Nout);
        if (route(p, false) == Route::kSmallTiles) assert(!pair_pays(p, 256));
        p.Nout = 1 << 22;
        assert(!pair_pays(p, 256));
    }
    // weights that one tile reads: few touched, neither layer's come as streaming loads, then the first's, then both
    const double mb = 1 << 20;
    assert(!stream_weights(false, 39 * mb) && stream_weights(false, 41 * mb) && !stream_weights(true, 79 * mb) && stream_weights(true, 81 * mb));
    assert(touched_weights(1, 2, 16, 16.0) == 2.0 && touched_weights(100000, 1, 4, 100.0) == 100.0 && touched_weights(3, 4, 4, 8.0) == 8.0);
    assert(std::abs(touched_weights(8, 2, 16, 16.0) - 16 * (1 - std::pow(0.875, 8))) < 1e-12);
    return 0;
}
"""


def test_both_sides_of_the_lines(tmp_path):
    (tmp_path / "routes.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++20", "-I" + os.path.join(ROOT, "paper_2103_13262_amd", "csrc"), str(tmp_path / "routes.cpp"), "-o", str(tmp_path / "routes")], check=True)
    subprocess.run([str(tmp_path / "routes")], check=True)
