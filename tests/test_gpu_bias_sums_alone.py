"""moe_bias_backward with either gradient left out: the other one as with both, nothing else written."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,d,h,E", [(300, 544, 96, 5), (40, 32, 2080, 300)])
def test_one_of_the_two(N, d, h, E, dtype):
    import torch

    print(f"[case] N {N} d {d} h {h} E {E} {dtype}", flush=True)
    dev = torch.device("cuda:0")
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev)
    g.manual_seed(N)
    X, Wg = (torch.empty(s, dtype=act, device=dev).normal_(generator=g) for s in ((N, d), (d, E)))
    desc = B.make_desc(N, d, h, E, 2, B.MOE_BF16 if dtype == "bf16" else B.MOE_F32, B.MOE_F32)
    buf = B.MoeLayerBuffers(desc, dev)
    ws = (buf.workspace, buf.ws_bytes, buf.stream())
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws)
    for name in ("dZ", "dYs"):
        off, n = B.moe_workspace_region(desc, name)
        buf.workspace[off:off + n].view(act).normal_(generator=g)
    new = lambda: [torch.full((E, w), 7.0, device=dev) for w in (h, d)]
    both, first, second = new(), new(), new()
    B.moe_bias_backward(desc, buf.plan, *both, *ws)
    B.moe_bias_backward(desc, buf.plan, first[0], None, *ws)
    B.moe_bias_backward(desc, buf.plan, None, second[1], *ws)
    B.moe_bias_backward(desc, buf.plan, None, None, *ws)
    assert torch.equal(first[0], both[0]) and torch.equal(second[1], both[1])
    assert bool((first[1] == 7.0).all()) and bool((second[0] == 7.0).all())
