"""GPU: the quantile kernel at the ends of its sorting networks (multiples of
eight states, then two runs of 128) and of its 2048-site chunks, against
numpy's sort of the same states, bit for bit."""
import numpy as np
import pytest

import paper_1811_01604_amd as mpr

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 2, 7, 8, 9, 16, 17, 40, 49, 64, 65, 100, 104, 105, 121, 128, 129, 200, 255, 256])
@pytest.mark.parametrize("ny,nx,p", [(1, 3, 0.5), (32, 64, 1.0), (41, 50, 0.5), (70, 90, 0.03)])
def test_quantiles_equal_sorted_states(M, ny, nx, p):
    rng = np.random.default_rng(M * 1000 + nx)
    n = ny * nx
    st = (rng.integers(0, 40, size=(M, n)) * 0.1570796 + rng.random((M, n)) * (rng.random(n) < 0.7)).astype(np.float32)
    z = rng.normal(50, 10, size=n).astype(np.float32)
    mask = (rng.random(n) >= p).astype(np.uint8)
    probs = np.array([0.0, 0.05, 0.37, 0.5, 0.95, 1.0])
    lo, hi = 12.5, 97.25
    ctx = mpr.Context(0)
    out = torch.zeros(probs.size * n, device="cuda")
    ctx.quantiles(mpr.images([(ny, nx)]), torch.from_numpy(z).cuda(), torch.from_numpy(mask).cuda(),
                  torch.from_numpy(st.ravel()).cuda(), M, probs, np.array([lo, hi]), out)
    ctx.close()
    v = np.sort(st, axis=0).astype(np.float64)
    for q, pr in enumerate(probs):
        h = (M - 1) * pr
        a = int(np.floor(h))
        phi = v[a] if a >= M - 1 else v[a] + (h - a) * (v[a + 1] - v[a])
        t = phi / (2.0 * np.pi)
        want = np.where(mask != 0, z, (lo * (1.0 - t) + hi * t).astype(np.float32))
        got = out[q * n:(q + 1) * n].cpu().numpy()
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), (q, pr)


@pytest.mark.parametrize("M,ny,nx,p", [(40, 2917, 2903, 0.5), (100, 2051, 2049, 0.5), (100, 2051, 2049, 0.04),
                                       (104, 1033, 1021, 0.9), (128, 1801, 1777, 0.5), (129, 521, 509, 0.5),
                                       (129, 521, 509, 0.04), (256, 307, 499, 0.9)])
def test_quantiles_of_many_sites(M, ny, nx, p):
    """Sizes at which a wave works along more than 64 sites, and (all but the
    104 and 256 states) along 320: gaps carried over from one group of 256
    sites to the next, full lists with a remainder, and the last few gaps.
    Every site, against a sort of the same states, bit for bit."""
    n = ny * nx
    g = torch.Generator(device="cuda").manual_seed(M + nx)
    st = 6.28 * torch.rand((M, n), generator=g, device="cuda")
    z = torch.randn(n, generator=g, device="cuda")
    mask = (torch.rand(n, generator=g, device="cuda") >= p).to(torch.uint8)
    probs = np.array([0.0, 0.37, 1.0])
    lo, hi = 12.5, 97.25
    ctx = mpr.Context(0)
    out = torch.full((probs.size, n), -1.0, device="cuda")
    ctx.quantiles(mpr.images([(ny, nx)]), z, mask, st.flatten(), M, probs, np.array([lo, hi]), out)
    ctx.close()
    for i in range(0, n, 1 << 20):
        v = torch.sort(st[:, i:i + (1 << 20)], dim=0).values.double()
        for q, pr in enumerate(probs):
            h = (M - 1) * pr
            a = int(np.floor(h))
            phi = v[a] if a >= M - 1 else v[a] + (h - a) * (v[a + 1] - v[a])
            t = phi / (2.0 * np.pi)
            j = slice(i, i + v.shape[1])
            want = torch.where(mask[j] != 0, z[j], (lo * (1.0 - t) + hi * t).float())
            assert torch.equal(out[q, j], want), (i, q)
