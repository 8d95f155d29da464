"""The gate's part of moe_backward (one launch, an expert's sums added up by the last of its workgroups to arrive) against
moe_scatter_backward on the same intermediates (two launches): bit for bit, since both add an expert's pieces of 64 rows in
ascending order.  Experts without rows, with one row, 64 and one more, and many pieces; one, two and several column blocks; more experts than a
wavefront has lanes and more than 256; each call twice (the counters are zero again after the first)."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,accumulate", [("bf16", 0), ("f32", 0), ("bf16", 1)])
@pytest.mark.parametrize("N,d,E,k", [(300, 32, 4, 2), (1, 576, 20, 1), (700, 1056, 70, 2), (900, 2080, 5, 3), (260, 1024, 300, 4), (40000, 32, 3, 2)])
def test_as_in_two_launches(N, d, E, k, dtype, accumulate):
    import torch

    print(f"[case] N {N} d {d} E {E} k {k} {dtype} accumulate {accumulate}", flush=True)
    dev, h = torch.device("cuda:0"), 32
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    dt = B.MOE_BF16 if dtype == "bf16" else B.MOE_F32
    grad = torch.float32 if accumulate else act
    g = torch.Generator(device=dev)
    g.manual_seed(N + d)
    new = lambda *s: torch.empty(s, dtype=act, device=dev).normal_(generator=g)
    X, Wg, dY, W1, W2 = new(N, d), new(d, E), new(N, d), new(E, d, h), new(E, h, d)
    bg = torch.linspace(12.0 * d ** 0.5, 0.0, E, device=dev)      # the last experts get no rows, the first nearly all
    desc = B.make_desc(N, d, h, E, k, dt, B.MOE_F32 if accumulate else dt, accumulate)
    buf = B.MoeLayerBuffers(desc, dev)
    ws = (buf.workspace, buf.ws_bytes, buf.stream())
    Y, dW1, dW2 = torch.empty_like(X), torch.zeros((E, d, h), dtype=grad, device=dev), torch.zeros((E, h, d), dtype=grad, device=dev)
    B.moe_plan(desc, X, Wg, bg, buf.plan, *ws)
    assert E == 4 or int(buf.counts[:E].min()) == 0
    B.moe_forward(desc, buf.plan, X, W1, W2, None, None, Y, *ws)

    def outputs():
        return torch.empty_like(X), torch.full((d, E), 0.5, dtype=grad, device=dev), torch.full((max(E, 4),), 0.5, device=dev)

    got = outputs()
    for _ in range(2):
        B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, *got, dW1, dW2, *ws)
    region = {}
    for name, dtp in (("Xs", act), ("dXs", act), ("dl", torch.float32)):
        off, n = B.moe_workspace_region(desc, name)
        region[name] = buf.workspace[off:off + n].view(dtp).clone()
    want = outputs()
    for _ in range(2):
        B.moe_scatter_backward(desc, buf.plan, Wg, region["Xs"], region["dXs"], region["dl"], *want, *ws)
    for a, b in zip(got, want):
        assert torch.equal(a[:E] if a.dim() == 1 else a, b[:E] if b.dim() == 1 else b)
