"""GPU: sweeps that keep their tiles on the chip (many per launch) against
one half-sweep launch at a time, bit for bit: double-precision chains, the
e(T, L) table chains, recorded states and tiles of 48 and 64 rows, at the
edges of the tiles (a single site wide, one tile, one row or column beyond a
tile, several ragged tiles)."""
import threading

import numpy as np
import pytest

import paper_1811_01604_amd as mpr
import synth

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    assert torch.cuda.is_available()
    c = mpr.Context(0)
    yield c
    c.close()


def image(ctx, ny, nx, p=0.6):
    z = torch.from_numpy(synth.matern_field(nx, ny, 0.5, 0.2, 50.0, 10.0, 3).astype(np.float32)).cuda().flatten()
    mk = torch.from_numpy(synth.random_mask(nx, ny, p, 4)).cuda().flatten()
    imgs = mpr.images([(ny, nx)])
    phi = torch.zeros_like(z)
    ctx.map_to_angles(imgs, z, mk, phi)
    return imgs, mk, phi


def run(ctx, imgs, phi, mk, T, tile, record=False, **kw):
    prm = mpr.default_params(tile_rows=tile, **kw)
    ws = torch.empty(ctx.workspace_size(imgs, prm), dtype=torch.uint8, device="cuda")
    ps = torch.zeros_like(phi)
    m2 = torch.zeros_like(phi) if prm.spread else None
    states = torch.zeros(prm.R * prm.K * phi.numel(), device="cuda") if record else None
    st = ctx.simulate(imgs, phi, mk, np.array([T]), prm, ws, ps, phi_m2=m2, phi_states=states)
    out = [ps, m2, states]
    return [o.cpu().numpy().tobytes() for o in out if o is not None], st


@pytest.mark.parametrize("fp64", [0, 1])
@pytest.mark.parametrize("ny,nx", [(2, 1), (1, 300), (8, 128), (9, 129), (33, 127), (65, 257), (200, 131)])
def test_resident_sweeps_equal_half_sweeps(ctx, ny, nx, fp64):
    """The tuned shape (a resident one at these sizes) with spread and
    recorded states, twice: the first call also tries the other shapes."""
    imgs, mk, phi = image(ctx, ny, nx) if ny * nx > 2 else (mpr.images([(2, 1)]),
                                                            torch.tensor([1, 0], dtype=torch.uint8, device="cuda"),
                                                            torch.tensor([1.0, 0.0], device="cuda"))
    for T in (2e-3, 0.05):
        kw = dict(R=3, K=5, spread=1, fp64=fp64, record=True)
        ref = run(ctx, imgs, phi, mk, T, 4, **kw)
        for _ in range(2):
            assert run(ctx, imgs, phi, mk, T, 0, **kw) == ref
        assert ctx.profile_read()["last_tile"] & mpr.TILE_PERSIST


@pytest.mark.parametrize("ny,nx", [(1500, 2048), (2048, 2047)])
def test_resident_tiles_of_48_and_64_rows(ctx, ny, nx):
    """Chains whose 32-row tiles do not fit on the GPU at once take 48 or 64 rows."""
    imgs, mk, phi = image(ctx, ny, nx)
    kw = dict(R=1, K=3, fixed_relax=6, spread=1)
    ref = run(ctx, imgs, phi, mk, 0.05, 48 | mpr.TILE_FUSED, **kw)
    assert run(ctx, imgs, phi, mk, 0.05, 32 | mpr.TILE_FUSED | mpr.TILE_PERSIST, **kw) == ref
    assert ctx.profile_read()["last_tile"] == 32 | mpr.TILE_FUSED | mpr.TILE_PERSIST


@pytest.mark.parametrize("q", [0.5, 0.25])
@pytest.mark.parametrize("ny,nx", [(1, 40), (16, 16), (70, 150), (257, 255)])
def test_resident_table_chains_equal_half_sweeps(ny, nx, q):
    """The temperature from table chains run in the tuned shapes and in the
    plain 4-row shape: the same energies, so the same number."""
    assert torch.cuda.is_available()
    got = []
    for tile in (4, 0):
        ctx = mpr.Context(0)
        imgs, mk, phi = image(ctx, ny, nx, 0.3)
        prm = mpr.default_params(tile_rows=tile, q=q, fp64=0 if q == 0.5 else 1, table_nT=8, table_T_lo=1e-4,
                                 table_T_hi=2.0, table_burn=40, table_meas=30)
        ws = torch.empty(ctx.workspace_size(imgs, prm), dtype=torch.uint8, device="cuda")
        e_s, T, cl = ctx.estimate_temperature(imgs, phi, mk, prm, ws)
        got.append((e_s[0], T[0], cl[0]))
        ctx.close()
    assert got[0] == got[1]


def test_a_short_wait_bound_does_not_end_other_calls(ctx):
    """A bound of 1 us on a block's wait holds for single-precision chains
    without recorded states; double precision, recorded states, table chains,
    tiles above 32 rows and the last chains of a larger set give the results
    of the default bound."""
    imgs, mk, phi = image(ctx, 512, 512)
    got = {}
    for bound in (0, 1):
        kw = dict(barrier_timeout_us=bound)
        tab = mpr.default_params(table_nT=8, table_T_lo=1e-4, table_T_hi=2.0, table_burn=40, table_meas=30, **kw)
        c = mpr.Context(0)  # (a table is kept by its context)
        ws = torch.empty(c.workspace_size(imgs, tab), dtype=torch.uint8, device="cuda")
        e_s, T, _ = c.estimate_temperature(imgs, phi, mk, tab, ws)
        big, big_mk, big_phi = image(c, 2048, 2047)
        got[bound] = (e_s[0], T[0], run(c, imgs, phi, mk, 0.05, 0, R=2, K=5, fp64=1, **kw),
                      run(c, imgs, phi, mk, 0.05, 0, R=2, K=5, record=True, **kw),
                      run(c, imgs, phi, mk, 0.05, 0, R=40, K=1, **kw),
                      run(c, big, big_phi, big_mk, 0.05, 0, R=1, K=3, fixed_relax=6, **kw))
        c.close()
    assert got[0] == got[1]


@pytest.mark.parametrize("fp64", [0, 1])
@pytest.mark.parametrize("p,ny,nx,R,rows,rows64", [
    (0.6, 61, 131, 16, 8, 8), (0.6, 61, 131, 20, 12, 12), (0.6, 61, 131, 30, 16, 16), (0.6, 61, 131, 40, 24, 24),
    (0.6, 61, 131, 60, 32, 32), (0.6, 61, 131, 70, 32, 24), (0.6, 47, 100, 150, 48, 16), (0.6, 61, 100, 150, 64, 24),
    (0.1, 61, 131, 5, 16, 16)])
def test_every_resident_tile_height(ctx, p, ny, nx, R, rows, rows64, fp64):
    """The number of chains and the share of gaps select the height of the
    tiles (of doubles, at most 32 rows): spread, recorded states and
    statistics against half-sweeps."""
    rows = rows64 if fp64 else rows
    imgs, mk, phi = image(ctx, ny, nx, p)
    kw = dict(R=R, K=4, spread=1, fp64=fp64, record=True)
    ref = run(ctx, imgs, phi, mk, 0.05, 4, **kw)
    assert run(ctx, imgs, phi, mk, 0.05, 0, **kw) == ref
    assert ctx.profile_read()["last_tile"] == min(rows, 32) | mpr.TILE_FUSED | mpr.TILE_PERSIST


def test_the_shape_does_not_depend_on_the_calls_before(ctx):
    """Two batches of six images with the same largest sides: the small one
    runs in resident tiles also after the large one, whose tiles do not fit,
    and the large one without them."""
    tiles = []
    for shapes in ([(1024, 1024)] * 6, [(1024, 1024)] + [(64, 64)] * 5) * 2:
        z = torch.from_numpy(np.concatenate([synth.matern_field(nx, ny, 0.5, 0.2, 50.0, 10.0, 3).astype(np.float32)
                                             .ravel() for ny, nx in shapes])).cuda()
        mk = torch.from_numpy(np.concatenate([synth.random_mask(nx, ny, 0.5, 4).ravel() for ny, nx in shapes])).cuda()
        imgs = mpr.images(shapes)
        phi, ps = torch.zeros_like(z), torch.zeros_like(z)
        ctx.map_to_angles(imgs, z, mk, phi)
        prm = mpr.default_params(R=1, K=50)
        ws = torch.empty(ctx.workspace_size(imgs, prm), dtype=torch.uint8, device="cuda")
        ctx.simulate(imgs, phi, mk, np.full(6, 0.05), prm, ws, ps)
        tiles.append(bool(ctx.profile_read()["last_tile"] & mpr.TILE_PERSIST))
    assert tiles == [False, True, False, True]


@pytest.mark.parametrize("own_streams", [False, True])
def test_threads_with_a_context_each(own_streams):
    """Three threads, each with its own context, on the default stream or on
    streams of their own: single precision, double precision and recorded
    states, with their e(T, L) tables, give the results of one thread."""
    jobs = [(side, kind) for side in (64, 300, 512, 1024) for kind in range(3)]

    def job(c, side, kind, stream):
        with torch.cuda.stream(stream):
            g = torch.Generator(device="cuda").manual_seed(side)
            z = 50 + 10 * torch.randn((side, side), generator=g, device="cuda")
            mk = (torch.rand((side, side), generator=g, device="cuda") >= 0.5).to(torch.uint8)
            imgs = mpr.images([(side, side)])
            phi, ps = torch.zeros_like(z), torch.zeros_like(z)
            c.map_to_angles(imgs, z, mk, phi, stream=stream)
            prm = mpr.default_params(R=2, K=20, fp64=1 if kind == 1 else 0, table_nT=8, table_burn=30, table_meas=30)
            ws = torch.empty(c.workspace_size(imgs, prm), dtype=torch.uint8, device="cuda")
            states = torch.zeros(40 * side * side, device="cuda") if kind == 2 else None
            e_s, T, _ = c.estimate_temperature(imgs, phi, mk, prm, ws, stream=stream)
            c.simulate(imgs, phi, mk, np.array([0.1]), prm, ws, ps, phi_states=states, stream=stream)
            stream.synchronize()
            return e_s[0], T[0], [o.cpu().numpy().tobytes() for o in (ps, states) if o is not None]

    c = mpr.Context(0)
    ref = [job(c, *j, torch.cuda.default_stream()) for j in jobs]
    c.close()
    wrong = []

    def worker(first):
        c = mpr.Context(0)
        stream = torch.cuda.Stream() if own_streams else torch.cuda.default_stream()
        for i in range(len(jobs)):
            k = (first + i) % len(jobs)
            try:
                if job(c, *jobs[k], stream) != ref[k]:
                    wrong.append((jobs[k], "differs"))
            except mpr.MprError as e:
                wrong.append((jobs[k], str(e)))
        c.close()

    threads = [threading.Thread(target=worker, args=(5 * t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


@pytest.mark.parametrize("fp64", [0, 1])
def test_launches_called_off_and_runs_resumed(ctx, fp64):
    """A bound of 1 us calls resident launches with recorded states off (their
    sweeps then run one launch each); runs of 11 sweeps a call, the first two
    of them so, the others resident, end as one run of half-sweeps does."""
    imgs, mk, phi = image(ctx, 130, 517)
    kw = dict(R=3, K=9, spread=1, fp64=fp64)
    ref = run(ctx, imgs, phi, mk, 0.05, 4, record=True, **kw)
    prm = mpr.default_params(sweep_limit=11, **kw)
    ws = torch.empty(ctx.workspace_size(imgs, prm), dtype=torch.uint8, device="cuda")
    ps, m2 = torch.zeros_like(phi), torch.zeros_like(phi)
    states = torch.zeros(prm.R * prm.K * phi.numel(), device="cuda")
    tiles, done = [], False
    while not done:
        prm.barrier_timeout_us = 1 if len(tiles) < 2 else 0
        prm.resume = 1 if tiles else 0
        done, st = ctx.simulate(imgs, phi, mk, np.array([0.05]), prm, ws, ps, phi_m2=m2, phi_states=states,
                                allow_incomplete=True)
        tiles.append(bool(ctx.profile_read()["last_tile"] & mpr.TILE_PERSIST))
    assert len(tiles) > 3 and not any(tiles[:2]) and all(tiles[2:])
    assert ([o.cpu().numpy().tobytes() for o in (ps, m2, states)], st) == ref
