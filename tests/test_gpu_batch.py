"""Batched persistent sweeps against the FP64 oracle run per simulation."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import batch_sweep
from tests.gpu_util import max_abs, require_gpu

pytestmark = pytest.mark.gpu

SHARED = dict(Du=0.2, Dv=0.1, dt=1.0)


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def _oracle(sim, i, n, noise=0.0, seed=0, side=12):
    shape = (sim.get("nz", sim.get("L")), sim.get("ny", sim.get("L")), sim.get("nx", sim.get("L")))
    u0, v0 = O.init_cube(shape=shape, side=side)
    return O.run(u0, v0, n, F=sim["F"], k=sim["k"], noise=noise, seed=seed + i, **SHARED)


def test_batch_mixed_sizes_bitwise(torch):
    """Uneven grids, own F and k each, noise keyed per simulation (seed + i);
    step counts that are not multiples of the fused depth."""
    from paper_2309_10292_amd import gs
    sims = [dict(nx=32, ny=32, nz=32, F=0.02, k=0.048), dict(nx=48, ny=40, nz=36, F=0.035, k=0.06),
            dict(nx=16, ny=20, nz=24, F=0.05, k=0.065), dict(nx=64, ny=24, nz=70, F=0.012, k=0.045)]
    for T in (1, 2, 3):
        for tile in gs.tblock_tiles():
            if T > gs.max_tblock(tile, "f64", batch=True):
                continue
            with gs.Batch(sims, noise=1e-3, seed=100, cube_side=8, tile=tile, tblock=T, zchunk=16, **SHARED) as b:
                b.step(7)
                for i, sm in enumerate(sims):
                    u, v = b.read(i)
                    ue, ve = _oracle(sm, i, 7, noise=1e-3, seed=100, side=8)
                    assert np.array_equal(u, ue) and np.array_equal(v, ve), (T, tile, i, max_abs(u, ue))


def test_batch_graph_and_tune(torch):
    """The autotuner picks a configuration per grid size without changing any
    state; graph replays (with eager steps between them) then match the oracle."""
    from paper_2309_10292_amd import gs
    sims = [dict(L=32, F=0.02, k=0.048), dict(L=48, F=0.03, k=0.055), dict(L=32, F=0.045, k=0.06),
            dict(L=64, F=0.025, k=0.05)]
    with gs.Batch(sims, cube_side=10, noise=1e-4, seed=5, **SHARED) as b:
        b.step(3)
        before = [b.read(i) for i in range(len(sims))]
        table = b.tune(reps=1)
        assert {(e["nx"], e["n_sims"]) for e in table} == {(32, 2), (48, 1), (64, 1)}
        for i in range(len(sims)):
            u, v = b.read(i)
            assert np.array_equal(u, before[i][0]) and np.array_equal(v, before[i][1])
        for rep in range(3):
            b.step_graph(5)
            b.step(1)
            torch.cuda.synchronize()
        for i, sm in enumerate(sims):
            u, v = b.read(i)
            ue, ve = _oracle(sm, i, 3 + 3 * 6, noise=1e-4, seed=5, side=10)
            assert np.array_equal(u, ue) and np.array_equal(v, ve), i


def test_batch_sweep_sample_bitwise(torch):
    """A sample of the (F, k) sweep's simulations (sizes 32..192) for 10
    steps, with the library's default configuration."""
    from paper_2309_10292_amd import gs
    sims = batch_sweep(12, seed=3)
    with gs.Batch(sims, **SHARED) as b:
        b.step(10)
        for i in (0, 5, 11):
            u, v = b.read(i)
            ue, ve = _oracle(sims[i], i, 10)
            assert np.array_equal(u, ue) and np.array_equal(v, ve), i
        d = b.diagnostics(3)
        e = O.diagnostics(*_oracle(sims[3], 3, 10))
        assert abs(d["sum_u"] - e["sum_u"]) <= 1e-13 * abs(e["sum_u"])


# tile 6 takes 64-, 48- and 32-cell tiles in one launch: grids of all three widths, ragged rows, chunks that do not
# divide them, and step counts split over launches of two depths
@pytest.mark.parametrize("T", [1, 2, 3])
@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "f16"])
def test_batch_tile_widths(torch, storage, T):
    """Every simulation equals the same one alone (single-grid results do not depend on the launch), bit for bit."""
    from paper_2309_10292_amd import gs
    sims = [dict(nx=80, ny=80, nz=20, F=0.03, k=0.06), dict(nx=48, ny=61, nz=18, F=0.035, k=0.06),
            dict(nx=24, ny=100, nz=17, F=0.02, k=0.05), dict(nx=128, ny=50, nz=19, F=0.04, k=0.06),
            dict(nx=72, ny=96, nz=9, F=0.012, k=0.045)]
    shared = dict(noise=1e-3, storage=storage, cube_side=8, **SHARED)
    with gs.Batch(sims, seed=50, tile=6, tblock=T, zchunk=8, **shared) as b:
        b.step(7)
        for i, sm in enumerate(sims):
            with gs.Sim(sm["nx"], sm["ny"], sm["nz"], F=sm["F"], k=sm["k"], seed=50 + i, **shared) as s:
                s.step(7)
                for got, want in zip(b.read(i), s.read()):
                    assert np.array_equal(got, want), (i, max_abs(got, want))


# the library's choice: every tile and depth it takes, chunks that do not divide the grids, grids of one chunk, and a
# chunk that the caller sets
@pytest.mark.parametrize("n,dims,storage,noise,zchunk,want", [
    (6, (32, 32, 32), "f64", 1e-3, 0, (5, 2)), (27, (40, 40, 40), "f64", 0.0, 0, (5, 2)),
    (32, (128, 128, 48), "f64", 0.0, 0, (6, 3)), (16, (80, 80, 80), "f32", 0.0, 0, (6, 2)),
    (7, (48, 40, 30), "f32", 1e-3, 0, (5, 2)), (20, (104, 90, 60), "bf16", 0.0, 0, (6, 2)),
    (5, (64, 64, 24), "f16", 0.0, 0, (5, 3)), (5, (64, 64, 24), "f16", 1e-3, 0, (5, 2)), (3, (24, 9, 5), "f32", 1e-3, 0, None),
    (4, (136, 31, 70), "f64", 1e-3, 11, None)])
def test_batch_library_choice(torch, n, dims, storage, noise, zchunk, want):
    """The tile and depth of the least estimated time, and the first and the last simulation bit for bit as alone."""
    from paper_2309_10292_amd import gs
    nx, ny, nz = dims
    sims = [dict(nx=nx, ny=ny, nz=nz, F=0.02 + 0.001 * i, k=0.055) for i in range(n)]
    shared = dict(noise=noise, storage=storage, cube_side=5, **SHARED)
    with gs.Batch(sims, seed=9, zchunk=zchunk, **shared) as b:
        c = b.config(0)
        assert want is None or (c["tile"], c["tblock"]) == want, c
        assert not zchunk or c["zchunk"] == zchunk
        b.step(8)
        for i in (0, n - 1):
            with gs.Sim(nx, ny, nz, F=sims[i]["F"], k=sims[i]["k"], seed=9 + i, **shared) as s:
                s.step(8)
                for got, one in zip(b.read(i), s.read()):
                    assert np.array_equal(got, one), (i, max_abs(got, one))


@pytest.mark.parametrize("dt", [1.0, 0.5])
@pytest.mark.parametrize("n", [4, 5])
def test_batch_three_steps_in_256_lanes(torch, n, dt):
    """FP64 without noise in the 256-lane tile: 256 work items of 8 planes, all resident, and 320, whose kernel does
    without straight-line levels; bit for bit the single grids."""
    from paper_2309_10292_amd import gs
    sims = [dict(L=64, F=0.02 + 0.005 * i, k=0.05 + 0.002 * i) for i in range(n)]
    shared = dict(Du=0.2, Dv=0.1, dt=dt, cube_side=20)
    with gs.Batch(sims, tile=5, tblock=3, zchunk=8, **shared) as b:
        b.step(7)
        got = [b.read(i) for i in range(n)]
    for i, sm in enumerate(sims):
        with gs.Sim(64, 64, 64, F=sm["F"], k=sm["k"], tile=2, **shared) as s:
            s.step(7)
            u, v = s.read()
        assert np.array_equal(got[i][0], u) and np.array_equal(got[i][1], v), i
