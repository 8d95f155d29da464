"""Sums over an expert's rows (expert-bias gradients, gate-matrix gradient) where the kernel changes over: a wavefront of eight rows
that has none, one, two, three and all of them, a piece of 64 rows with one more row, experts without rows, and both searches for
a piece's expert (up to 256 experts and more), one, two and several column blocks (whose order changes), and more pieces than one grid
dimension holds.  All numbers are small integers, so every sum is exact."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 3, 8, 9, 10, 11, 0, 63, 64, 65, 66, 67, 128, 130]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("E,d,h", [(16, 32, 1056), (256, 256, 32), (257, 288, 544), (700, 704, 32), (16, 2080, 640), (4, 32, 32)])
def test_sums_over_segments(E, d, h, dtype):
    import torch

    print(f"[case] E {E} d {d} h {h} {dtype}", flush=True)
    dev = torch.device("cuda:0")
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev)
    g.manual_seed(E + h)
    rows = EDGES if E == 16 else [2100000, 0, 130, 7] if E == 4 else [(0, 1, 0, 2, 11, 1, 0, 3)[e % 8] + (130 if e == E - 1 else 0) for e in range(E)]
    N = sum(rows)
    expert = torch.repeat_interleave(torch.arange(E, device=dev), torch.tensor(rows, device=dev))[torch.randperm(N, generator=g, device=dev)]
    X, Wg = torch.zeros((N, d), dtype=act, device=dev), torch.zeros((d, E), dtype=act, device=dev)
    X[torch.arange(N, device=dev), expert] = 1     # one feature per expert decides: the experts' row counts are exact
    Wg[torch.arange(E), torch.arange(E)] = 1
    desc = B.make_desc(N, d, h, E, 1, B.MOE_BF16 if dtype == "bf16" else B.MOE_F32, B.MOE_F32)
    buf = B.MoeLayerBuffers(desc)
    ws = (buf.workspace, buf.ws_bytes, buf.stream())
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws)
    assert buf.counts[:E].tolist() == rows

    def region(name, width):
        off, n = B.moe_workspace_region(desc, name)
        t = buf.workspace[off:off + n].view(act).view(N, width)
        return t.copy_(torch.randint(-8, 9, (N, width), generator=g, device=dev))

    def sums(rows_of, weights=None):
        r = rows_of.double() if weights is None else rows_of.double() * weights.double()[:, None]
        return torch.stack([s.sum(0) for s in r.split(rows)])

    dZ, dYs = region("dZ", h), region("dYs", d)
    db1, db2 = (torch.full((E, w), float("nan"), device=dev) for w in (h, d))
    B.moe_bias_backward(desc, buf.plan, db1, db2, *ws)
    assert torch.equal(db1.double(), sums(dZ)) and torch.equal(db2.double(), sums(dYs))

    Xs, dXs = (torch.randint(-8, 9, (N, d), generator=g, device=dev).to(act) for _ in range(2))
    dl = torch.randint(-8, 9, (N,), generator=g, device=dev).float()
    dX, dWg, dbg = torch.empty_like(X), torch.full((d, E), float("nan"), device=dev), torch.full((max(E, 4),), float("nan"), device=dev)
    B.moe_scatter_backward(desc, buf.plan, Wg, Xs, dXs, dl, dX, dWg, dbg, *ws)
    by_row = dl[buf.perm[:N].long()]
    assert torch.equal(dWg.double(), sums(Xs, by_row).T) and torch.equal(dbg[:E].double(), sums(torch.ones((N, 1), device=dev), by_row)[:, 0])
