"""The rule that says which workgroups take the experts' last pieces, at the shapes whose results test_gpu_last_pieces.py checks:
their comment says which side of the line each of them is on.  (The rule's header is compiled for the host.)"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cassert>
#include "last_pieces.h"
using namespace moe;

int main()
{
    const int W = 32, columns = 4;          // 256 workgroups; dXs of d = 1024 in tiles 256 wide
    struct { int blocks, pieces, free; bool stay; } shapes[] = {{62, 20, 1, false}, {56, 16, 4, true}, {56, 17, 4, false}, {64, 9, 32, true}};
    for (auto& s : shapes) {
        const int first = first_free_workgroup((long)s.blocks * columns, W);
        assert(W - first == s.free);
        assert(last_pieces_stay((long)s.pieces * columns, first, W) == s.stay);
    }
    // a round that is full leaves nobody free and the next begins with the first workgroup; one tile more takes one of each XCD's
    assert(first_free_workgroup(8L * W, W) == 0 && first_free_workgroup(8L * W + 1, W) == 1 && first_free_workgroup(8L * W - 8, W) == W - 1);
    for (int first = 0; first < W; ++first)
        assert(last_pieces_stay(16L * (W - first), first, W) && !last_pieces_stay(16L * (W - first) + 1, first, W));
    return 0;
}
"""


def test_two_last_pieces_stay_with_a_free_workgroup(tmp_path):
    source, program = tmp_path / "rule.cpp", tmp_path / "rule"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++20", "-I" + os.path.join(ROOT, "paper_2103_13262_amd", "csrc"), str(source), "-o", str(program)], check=True)
    subprocess.run([str(program)], check=True)
