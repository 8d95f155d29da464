"""H and dZ over all of GeLU's range, in the small tiles (few rows) and in the persistent kernels: no weights in front of the
pre-activations (they are the bias) nor behind them (dH is 1), against 64 bits."""
import pytest

from paper_2103_13262_amd import binding as B

pytestmark = pytest.mark.gpu


# a handful of rows: both products in the small tiles; 8192 rows of one expert: both in the persistent kernels, which look the factors up
@pytest.mark.parametrize("N,small", [(40, True), (8192, False)])
def test_every_pre_activation(N, small):
    import torch

    dev, d = torch.device("cuda:0"), 2048
    bits = torch.arange((127 - 14) << 7, ((127 + 3) << 7) + 33, dtype=torch.int32)        # 2^-14 to 8 and a quarter, and their negatives
    z = torch.cat([(bits << 16).view(torch.float32), -(bits << 16).view(torch.float32)])
    z = torch.nn.functional.pad(z, (0, -len(z) % 32)).to(dev)
    h = len(z)
    print(f"[case] N {N} d {d} h {h}", flush=True)
    new = lambda shape: torch.zeros(shape, dtype=torch.bfloat16, device=dev)
    X, Wg, W1, W2, dY = new((N, d)), new((d, 1)), new((1, d, h)), new((1, h, d)), new((N, d))
    W2[0, :, 0], dY[:, 0] = 1, 1
    b1, b2 = z.bfloat16()[None].contiguous(), new((1, d))
    desc = B.make_desc(N, d, h, 1, 1)
    buf = B.MoeLayerBuffers(desc, dev)
    ws, st = (buf.workspace, buf.ws_bytes), buf.stream()
    Y, dX, dWg, dW1, dW2 = (torch.empty_like(t) for t in (dY, X, Wg, W1, W2))
    B.moe_plan(desc, X, Wg, None, buf.plan, *ws, st)
    B.moe_forward(desc, buf.plan, X, W1, W2, b1, b2, Y, *ws, st)
    B.moe_backward(desc, buf.plan, X, Wg, W1, W2, dY, dX, dWg, torch.empty(4, device=dev), dW1, dW2, *ws, st)

    def region(name):
        off, n = B.moe_workspace_region(desc, name)
        return buf.workspace[off:off + n].view(torch.bfloat16).view(N, h)

    Z, H, dZ = region("Z"), region("H"), region("dZ")
    assert torch.equal(Z[0], b1[0])
    for t in (Z, H, dZ):
        assert torch.equal(t, t[:1].expand_as(t))
    v = z.double()
    cdf = 0.5 * torch.erfc(-v / 2 ** 0.5)
    slope = cdf + v * torch.exp(-0.5 * v * v) / (2 * torch.pi) ** 0.5
    # rounding to 8 significant bits: 2^-8 of the value (half a unit, at most); the factor in 32 bits is off by less than 1e-5 of Phi (the power's
    # argument is rounded), the derivative by 1.3e-7; outside 2^-11 .. 8 a table's nearest entry is off by less than 4e-4
    outside = ((v.abs() < 2 ** -11) | (v.abs() >= 8)).double() * (0 if small else 4e-4)
    for name, got, ref, off in (("H", H[0], v * cdf, v.abs() * (1e-5 * cdf + outside)), ("dZ", dZ[0], slope, 1.3e-7 + outside)):
        over = (got.double() - ref).abs() - (2.0 ** -8 * ref.abs() * (1 + 1e-5) + off * (1 + 2.0 ** -8))
        assert float(over.max()) <= 0, (name, float(v[over.argmax()]), float(got[over.argmax()]), float(ref[over.argmax()]))
