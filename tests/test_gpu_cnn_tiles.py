"""GPU: the weight-gradient kernel at the edges of its 16 x 32-pixel tiles and
of its 256 persistent blocks, against a float64 correlation."""
import numpy as np
import pytest

import paper_1811_01604_amd as mpr

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
C, WSZ = 32, 9 * 32 * 32


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (1, 16, 32), (1, 17, 33), (3, 15, 31), (1, 3, 70), (2, 100, 5),
                                   (1, 260, 520), (5, 130, 97)])
def test_weight_gradient(n, h, w, masked):
    """Products of bfloat16 values are exact in single precision, so a sum of
    N of them, in any order, is within N 2^-24 sum |x g| of its exact value
    (255 blocks of partial sums more at most)."""
    ctx = mpr.Context(0)
    gen = torch.Generator(device="cuda").manual_seed(n * 7919 + h * 131 + w)
    x, g, ref = (torch.randn((n, h, w, C), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    grads = torch.full((WSZ + C,), float("nan"), device="cuda")
    ws = torch.empty(256 * 4 * (WSZ + C) * 4, dtype=torch.uint8, device="cuda")
    ctx.cnn_diag_wgrad(x, g, grads, ws, gref=ref if masked else None)
    ctx.close()
    g64 = (g.double() * (ref > 0) if masked else g.double()).cpu().numpy().reshape(-1, C)
    xp = np.pad(x.double().cpu().numpy(), ((0, 0), (1, 1), (1, 1), (0, 0)))
    got = grads.double().cpu().numpy()
    eps = (n * h * w + 256) * 2.0 ** -24
    for t in range(9):
        xs = xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(-1, C)
        bound = eps * (np.abs(xs).T @ np.abs(g64)) + 1e-30
        err = np.abs(got[t * C * C:(t + 1) * C * C].reshape(C, C) - xs.T @ g64)
        assert (err <= bound).all(), (t, float((err / bound).max()))
    err = np.abs(got[WSZ:] - g64.sum(0))
    assert (err <= eps * np.abs(g64).sum(0) + 1e-30).all()


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (1, 16, 32), (1, 17, 33), (3, 15, 31), (2, 100, 5), (5, 130, 97),
                                   (1, 260, 520), (3, 330, 520)])
def test_weight_gradient_of_integers(n, h, w, masked):
    """Integers of at most 2: every product and partial sum is a whole number
    below 2^24, so the sums are exact in single precision in any order, and a
    pixel left out or counted twice shows.  Up to 1071 tiles, four or five for
    each of the 256 blocks."""
    ctx = mpr.Context(0)
    rng = np.random.default_rng(n * 7919 + h * 131 + w)
    x, g = (rng.integers(-2, 3, size=(n, h, w, C)) for _ in range(2))
    ref = rng.normal(size=(n, h, w, C))
    xd, gd, rd = (torch.from_numpy(a).to(torch.bfloat16).cuda() for a in (x, g, ref))
    grads = torch.full((WSZ + C,), float("nan"), device="cuda")
    ws = torch.empty(256 * 4 * (WSZ + C) * 4, dtype=torch.uint8, device="cuda")
    ctx.cnn_diag_wgrad(xd, gd, grads, ws, gref=rd if masked else None)
    ctx.close()
    gm = (g * (ref > 0) if masked else g).reshape(-1, C).astype(np.float64)
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0))).astype(np.float64)
    want = [(xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(-1, C).T @ gm).ravel() for t in range(9)]
    assert np.array_equal(grads.double().cpu().numpy(), np.concatenate(want + [gm.sum(0)]))
