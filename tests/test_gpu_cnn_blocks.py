"""GPU: the residual-block kernel of the network against single convolutions,
bit for bit, and on very wide images."""
import pytest

import paper_1811_01604_amd as mpr

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    assert torch.cuda.is_available()
    c = mpr.Context(0)
    yield c
    c.close()


def random_network(ctx, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = 0.06 * torch.randn(ctx.cnn_param_count(), generator=g, device="cuda")
    packed = torch.empty(ctx.cnn_packed_bytes() // 2, dtype=torch.bfloat16, device="cuda")
    ctx.cnn_pack(p, packed)
    return p, packed


def infer(ctx, p, packed, phi, mask):
    n, h, w = phi.shape
    ws = torch.empty(ctx.cnn_workspace_size(n, h, w, False), dtype=torch.uint8, device="cuda")
    out = torch.full_like(phi, -1.0)
    ctx.cnn_infer(p, packed, phi, mask, ws, out)
    torch.cuda.synchronize()
    return out


def test_rows_of_eight_million_pixels(ctx):
    """The 18 rows around a tile span more than 2^32 activations here.  An
    output depends on the 18 pixels around it (18 layers of 3 x 3), so columns
    of the wide image equal those of a narrow cut around them bit for bit."""
    h, w, cut, rim = 30, 7_900_030, 300, 20
    p, packed = random_network(ctx, 5)
    g = torch.Generator(device="cuda").manual_seed(6)
    phi = 6.28 * torch.rand((1, h, w), generator=g, device="cuda")
    mask = (torch.rand((1, h, w), generator=g, device="cuda") < 0.5).to(torch.uint8)
    wide = infer(ctx, p, packed, phi, mask)
    for c0 in (0, 1_000_001, w - cut):
        lo, hi = (0 if c0 == 0 else rim), (cut if c0 == w - cut else cut - rim)
        narrow = infer(ctx, p, packed, phi[:, :, c0:c0 + cut].contiguous(), mask[:, :, c0:c0 + cut].contiguous())
        assert torch.equal(wide[:, :, c0 + lo:c0 + hi], narrow[:, :, lo:hi]), c0


@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (1, 14, 30), (1, 15, 31), (2, 37, 61), (1, 29, 200), (3, 251, 389)])
def test_forward_equals_single_convolutions(ctx, n, h, w):
    """Both modes of the forward pass run a residual block as one kernel, the
    inner activation in LDS; the training mode also keeps it for the backward
    pass.  Reference: one launch per convolution on the same packed weights.
    The output of either mode and every kept activation have the same bits, on
    shapes around the kernel's 14 x 30 output tile and with more tiles (702)
    than the GPU holds blocks (512)."""
    WSZ, B = 9 * 32 * 32, 8
    p, packed = random_network(ctx, h)
    p.view(2 * B + 2, WSZ + 32)[:, WSZ:] *= 5.0  # (biases that reach the rounding)
    g = torch.Generator(device="cuda").manual_seed(w)
    x = torch.randn((n, h, w, 32), generator=g, device="cuda").to(torch.bfloat16)

    def conv(k, src, add=None, relu=False):
        out = torch.empty_like(src)
        ctx.cnn_diag_conv(src, packed[2 * k * WSZ:(2 * k + 1) * WSZ], p[k * (WSZ + 32) + WSZ:(k + 1) * (WSZ + 32)], out,
                          add=add, relu=relu)
        return out

    hs, ts = [conv(0, x, relu=True)], []
    for b in range(B):
        ts.append(conv(1 + 2 * b, hs[-1], relu=True))
        hs.append(conv(2 + 2 * b, ts[-1], add=hs[-1]))
    want = conv(2 * B + 1, hs[-1])
    assert (ts[-1] > 0).any() and (ts[-1] == 0).any()
    for training in (False, True):
        ws = torch.empty(ctx.cnn_workspace_size(n, h, w, training), dtype=torch.uint8, device="cuda")
        y = torch.full_like(x, -3.0)
        ctx.cnn_forward(p, packed, x, ws, y, training=training)
        assert torch.equal(y.view(torch.int16), want.view(torch.int16)), training
    # the training workspace: the nine block inputs, then the eight inner
    # activations, each rounded up to 256 bytes
    size = x.numel() * 2
    for k, t in enumerate(hs + ts):
        at = k * ((size + 255) // 256 * 256)
        assert torch.equal(ws[at:at + size].view(torch.int16), t.view(torch.int16).flatten()), k
