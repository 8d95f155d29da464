"""The persistent kernels' products (two size classes of rows, and the pairs of the backward pass) with ragged widths, gathered rows, biases and last
pieces of all lengths: whole matrices against torch in fp32.  Which kernel each case reaches is stated and checked against the rule
itself (compiled for the host), so that a new line cannot take the cases elsewhere unnoticed."""
import os
import subprocess

import pytest

from paper_2103_13262_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# d, h, experts' rows, top-k, biases.  Widths end 64-deep blocks at 32 and 128-deep ones at 32 and 96, and fill neither 256 nor 512 columns.
# The first layer's reduction is d, the second's h; below 2048 a reduction is shallow: it is never cut, and few last pieces run in tiles with
# 128-deep blocks, many in 128 x 512 ones; from 2048 on, tiles are cut along it.
CASES = {
    "shallow_and_cut": (1120, 2080, [256 * 4 + 1, 256 * 5 + 127, 256 * 3 + 128, 256 * 5 + 129, 256 * 6, 256 * 3 + 31], 2, True),
    "cut_and_shallow": (2080, 2016, [256 * 7 + 33, 256 * 6 + 64, 256 * 5 + 255, 256 * 8 + 2, 256 * 6 + 97], 1, False),
    "many_last_pieces": (1120, 2080, [256 + 5 * e + 1 for e in range(20)], 2, True),
    "last_pieces_only": (1120, 2080, [72 + e for e in range(56)] + [128] * 8, 2, False),
    "whole_blocks_only": (1120, 2080, [256 * 5, 256 * 6, 256 * 4, 256 * 5, 256 * 7], 1, True),
    "rounds_then_last_pieces": (1120, 2080, [256 * 9 + 40, 256 * 10 + 100, 256 * 8 + 7, 256 * 11 + 128, 256 * 9 + 1, 256 * 9 + 60], 2, False),
}

ROUTES = r"""
#include <cassert>
#include "routes.h"
using namespace moe;
struct Product { long M; int E, K, Nout, stream_out, accumulate, out_f32, wide_gather; };
int main()
{
    const Product cases[] = {%s};
    for (const Product& fc1 : cases) {
        Product fc2 = fc1;
        fc2.K = fc1.Nout; fc2.Nout = fc1.K;
        for (const Product& p : {fc1, fc2})
            for (bool forward : {true, false}) assert(route(p, forward) == Route::kClasses);
        Product far = fc1;       // the same layer with its rows gathered from 4 GB and more
        far.wide_gather = 1;
        assert(route(far, true) == Route::kWideClasses);
        // dZ runs over d with h columns, dXs over h with d columns, each beside a weight gradient
        assert(pair_pays(fc1, 256) && pair_pays(fc2, 256));
    }
    return 0;
}
"""


def test_the_cases_reach_the_kernels_they_are_for(tmp_path):
    sizes = ["{%d, %d, %d, %d, %d, 0, 0, 0}" % (sum(rows), len(rows), d, h, len(rows) * d * h * 2 > 48 << 20) for d, h, rows, _, _ in CASES.values()]
    (tmp_path / "routes.cpp").write_text(ROUTES % ", ".join(sizes))
    subprocess.run(["g++", "-std=c++20", "-I" + os.path.join(ROOT, "paper_2103_13262_amd", "csrc"), str(tmp_path / "routes.cpp"), "-o", str(tmp_path / "routes")], check=True)
    subprocess.run([str(tmp_path / "routes")], check=True)
    d, h, rows, _, _ = CASES["many_last_pieces"]     # too many for the 128-deep tiles in FC1; the others' fit one round of them
    columns = lambda width: (width + 127) // 128
    pieces = {n: sum(0 < r % 256 <= 128 for r in c[2]) for n, c in CASES.items()}
    assert pieces["many_last_pieces"] * columns(h) > 256 >= pieces["shallow_and_cut"] * columns(h)
    assert pieces["whole_blocks_only"] == 0 and max(CASES["last_pieces_only"][2]) == 128
    whole = lambda n: sum((r + 127) // 256 for r in CASES[n][2]) * ((CASES[n][0] + 255) // 256)      # FC2's big tiles: a round is 256
    assert whole("shallow_and_cut") < 256 <= whole("rounds_then_last_pieces")


def _routed(torch, N, d, rows, k, dev, gen):
    """X and W_g that send exactly rows[e] assignments to expert e: one feature per expert decides, the first choice's is larger."""
    E = len(rows)
    a = torch.repeat_interleave(torch.arange(E), torch.tensor(rows)).view(k, N)      # (sorted, so a token's choices differ: no expert has more than N rows)
    a = a[:, torch.randperm(N, generator=gen)].to(dev)
    X = torch.empty((N, d), dtype=torch.bfloat16, device=dev).normal_()
    X[:, :E] = 0
    for j in range(k):
        X[torch.arange(N, device=dev), a[j]] = 2.0 - j
    Wg = torch.zeros((d, E), dtype=torch.bfloat16, device=dev)
    Wg[torch.arange(E), torch.arange(E)] = 1
    return X, Wg


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_products(name):
    import torch

    d, h, rows, k, biases = CASES[name]
    E, M, dev = len(rows), sum(rows), torch.device("cuda:0")
    N = M // k
    assert M % k == 0 and max(rows) <= N
    print(f"[case] {name}: N {N} d {d} h {h} E {E} k {k}", flush=True)
    torch.manual_seed(E + M)
    gen = torch.Generator().manual_seed(E + M)
    X, Wg = _routed(torch, N, d, rows, k, dev, gen)
    normal = lambda shape, std: torch.empty(shape, dtype=torch.bfloat16, device=dev).normal_(0.0, std)
    W1, W2, dY = normal((E, d, h), 0.06), normal((E, h, d), 0.06), normal((N, d), 1.0)
    b1, b2 = (normal((E, h), 1.0), normal((E, d), 1.0)) if biases else (None, None)
    desc = B.make_desc(N, d, h, E, k)
    buf = B.MoeLayerBuffers(desc, dev)
    ws, st = (buf.workspace, buf.ws_bytes), buf.stream()
    Y, dX, dWg, dW1, dW2 = (torch.full_like(t, float("nan")) for t in (dY, X, Wg, W1, W2))
    dbg = torch.empty(max(E, 4), device=dev)
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
    B.moe_forward(desc, buf.plan, X, W1, W2, b1, b2, Y, *ws, st)
    assert buf.counts[:E].tolist() == rows

    def region(name, width):
        off, n = B.moe_workspace_region(desc, name)
        return buf.workspace[off:off + n].view(torch.bfloat16).view(M, width)

    # exact products; both sums round by at most depth * 2^-24 of the terms' size each, the result to bf16 by 2^-8 of itself; off: what else
    # the result may be off by
    def check(what, got, a, w, bias=None, factor=None, off=0.0):
        ref, size = a @ w, a.abs() @ w.abs()
        if bias is not None:
            ref, size = ref + bias.float(), size + bias.float().abs()
        f = torch.ones((), device=dev) if factor is None else factor
        bound = 2 * (a.shape[1] + 1) * 2.0 ** -24 * size * f.abs() + ref.abs() * (2.0 ** -8 * f.abs() * 1.01 + off) + 1e-30
        over = float(((got.float() - ref * f).abs() - bound).max())      # (a NaN fails too)
        assert over <= 0, (what, over)

    perm = buf.perm[:M].long()
    Z, H = region("Z", h), region("H", h)
    out = Y[perm // k] if k == 1 else region("Ys", d)
    outside = lambda z: (z.abs() < 2.0 ** -11) | (z.abs() >= 8)          # a table's nearest entry stands for these: off by less than 4e-4
    gauss = lambda z: torch.exp(-0.5 * z * z) / (2 * torch.pi) ** 0.5
    segments, r0 = [], 0
    for e, n in enumerate(rows):
        segments.append((e, slice(r0, r0 + n)))
        r0 += n
    for e, seg in segments:
        check(("Z", e), Z[seg], X[perm[seg] // k].float(), W1[e].float(), b1[e] if biases else None)
        check(("Ys", e), out[seg], H[seg].float(), W2[e].float(), b2[e] if biases else None)
        # H of a sum that rounds to Z lies between the function's values at both ends (its one minimum may lie between them); looked up at
        # Z and carried along the slope it is off by the second-order rest, |z| delta^2 / 2 times the largest |x| phi(x) between the ends
        z = Z[seg].double()
        delta = 2.0 ** -8 * z.abs()
        ends = torch.stack([z - delta, z + delta])
        ends = ends * 0.5 * torch.erfc(-ends / 2 ** 0.5)
        rest = 0.5 * z.abs() * delta ** 2 * (z.abs() + delta) * gauss(z.abs() - delta)
        slack = (2.0 ** -8 + 2e-5) * ends.abs().amax(0) + 1.01 * rest + outside(z) * z.abs() * 4e-4 + 1e-30
        between = torch.where((z + 0.752).abs() < 0.01, delta ** 2, torch.zeros_like(z))
        over = float(torch.maximum(H[seg].double() - ends.amax(0) - slack, ends.amin(0) - between - slack - H[seg].double()).max())
        assert over <= 0, ("H", e, over)

    # in pairs, then each product in a launch of its own (a gradient in the place of its weight must wait for the product that reads the weight)
    for in_place in (False, True):
        g1, g2 = (W1.clone(), W2.clone()) if in_place else (dW1, dW2)
        B.moe_backward(desc, buf.plan, X, Wg, g1 if in_place else W1, g2 if in_place else W2, dY, dX, dWg, dbg, g1, g2, *ws, st)
        dYs, dZ, dXs, Xs = region("dYs", d), region("dZ", h), region("dXs", d), region("Xs", d)
        for e, seg in segments:
            z = Z[seg].double()
            slope = (0.5 * torch.erfc(-z / 2 ** 0.5) + z * gauss(z)).float()
            check(("dZ", e), dZ[seg], dYs[seg].float(), W2[e].float().T, factor=slope, off=outside(z).float() * 4e-4 + 1.3e-7)
            check(("dXs", e), dXs[seg], dZ[seg].float(), W1[e].float().T)
            check(("dW1", e), g1[e], Xs[seg].float().T, dZ[seg].float())
            check(("dW2", e), g2[e], H[seg].float().T, dYs[seg].float())
    status = B.moe_check_status(desc, buf.workspace, buf.ws_bytes, st)
    assert status == 0
