"""GPU: the network input and the loss gradient at pixel counts around a
wave's 64 and a block's 256 pixels, against the float64 oracle; every channel
of every pixel is written and nothing behind the last one."""
import numpy as np
import pytest

import paper_1811_01604_amd as mpr
from oracle import cnn

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
C = 32


@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (1, 7, 9), (1, 8, 8), (1, 5, 13), (1, 1, 255), (1, 16, 16), (1, 1, 257),
                                   (3, 25, 39)])
def test_input_and_loss(n, h, w):
    """A value is rounded to bfloat16 once (a relative 2^-9) from a single
    precision one with an error of a few 2^-24."""
    rng = np.random.default_rng(n * 7919 + h * 131 + w)
    px = n * h * w
    phi = rng.uniform(0, 2 * np.pi, (n, h, w)).astype(np.float32)
    smp = (rng.random((n, h, w)) < 0.5).astype(np.uint8)
    target = rng.uniform(-1, 1, (n, h, w, 2)).astype(np.float32)
    y = torch.from_numpy(rng.normal(size=(n, h, w, C))).to(torch.bfloat16).cuda()
    big = torch.full((2, px * C + 4096), 7.0, dtype=torch.bfloat16, device="cuda")
    x, dy = (b[:px * C].view(n, h, w, C) for b in big)
    ctx = mpr.Context(0)
    sd = torch.from_numpy(smp).cuda()
    ctx.cnn_encode(torch.from_numpy(phi).cuda(), sd, x)
    gaps = int((smp == 0).sum())
    ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
    if gaps:
        got_loss = ctx.cnn_loss(y, torch.from_numpy(target).cuda(), sd, gaps, dy, ws)
    torch.cuda.synchronize()
    ctx.close()
    assert (big[0, px * C:] == 7.0).all() and (big[1, px * C:] == 7.0).all()
    want = cnn.encode(phi.astype(np.float64), smp)
    assert (np.abs(x.double().cpu().numpy() - want) <= 2.0 ** -8 * np.abs(want) + 1e-6).all()
    if gaps:
        loss, dwant = cnn.loss(y.double().cpu().numpy(), target.astype(np.float64), smp == 0)
        assert abs(got_loss - loss) <= 1e-5 * loss
        assert (np.abs(dy.double().cpu().numpy() - dwant) <= 2.0 ** -8 * np.abs(dwant) + 1e-6 / gaps).all()
