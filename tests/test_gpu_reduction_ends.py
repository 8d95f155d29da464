"""bf16 products whose reductions end inside a block of the main loop: what lies behind the end belongs to another expert and must
not reach the result, whatever it holds."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


# widths that end a 64-deep block in its middle, a 32-deep one at its end, a 128-deep one at each quarter; rows that end a 32-deep block at
# every kind of place (the weight gradients' reductions), in small tiles and pairs; the last case's forward products run in size classes
@pytest.mark.parametrize("d,h,rows", [(96, 160, [33, 1, 300, 70, 0, 130]), (32, 96, [16, 17, 40, 15, 31, 2]), (224, 2144, [257, 129, 600, 383, 8, 24]),
                                      (288, 64, [5, 6, 7, 9, 10, 11]), (2080, 96, [500, 270, 260, 390]),
                                      (1120, 2080, [1025, 1407, 896, 1409, 1536, 799])])
def test_the_next_experts_values_stay_out(d, h, rows):
    import torch

    print(f"[case] d {d} h {h} rows {rows}", flush=True)
    E, N, dev = len(rows), sum(rows), torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(d + h)
    normal = lambda shape, std=1.0: torch.empty(shape, dtype=torch.bfloat16, device=dev).normal_(0.0, std, generator=g)
    expert = torch.repeat_interleave(torch.arange(E, device=dev), torch.tensor(rows, device=dev))[torch.randperm(N, generator=g, device=dev)]
    X, Wg = normal((N, d)), torch.zeros((d, E), dtype=torch.bfloat16, device=dev)
    X[:, :E] = 0                                   # one feature per expert decides: the experts' row counts are exact
    X[torch.arange(N, device=dev), expert] = 1
    Wg[torch.arange(E), torch.arange(E)] = 1
    W1, W2, dY = normal((E, d, h), 0.05), normal((E, h, d), 0.05), normal((N, d))
    desc = B.make_desc(N, d, h, E, 1)
    buf = B.MoeLayerBuffers(desc, dev)
    ws, st = (buf.workspace, buf.ws_bytes), buf.stream()

    def run():
        Y, dX, dWg, dW1, dW2 = (torch.empty_like(t) for t in (dY, X, Wg, W1, W2))
        B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
        B.moe_forward(desc, buf.plan, X, W1, W2, None, None, Y, *ws, st)
        B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, dX, dWg, torch.empty(max(E, 4), device=dev), dW1, dW2, *ws, st)
        assert buf.counts[:E].tolist() == rows
        return Y, dX, dW1, dW2

    clean = run()
    bad = 2                                        # this expert's weights, and with them its rows of Z, H, dZ, are not finite
    W1[bad], W2[bad] = float("inf"), float("nan")
    other_rows, other = expert != bad, [e for e in range(E) if e != bad]
    for name, a, b in zip(("Y", "dX", "dW1", "dW2"), clean, run()):
        pick = other_rows if name in ("Y", "dX") else other
        assert torch.equal(a[pick], b[pick]), name
        assert bool(a[pick].isfinite().all()), name
